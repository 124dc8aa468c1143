"""RANSAC at the edges of its tiles (16 attempts a tile, 64, 128 or 256 a
workgroup, blocks of 64 points): every attempt and result equals the oracle."""
import numpy as np
import pytest

from paper_2210_14771_amd import api

import test_gpu_parity as parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _frames(n, W, H, seed):
    """A noisy disc on a noisy dark border; every third frame all noise near
    one edge (nearly straight lines of candidates)."""
    rng = np.random.default_rng(seed)
    yy, xx = np.mgrid[0:H, 0:W]
    out = np.empty((n, H, W, 3), dtype=np.uint8)
    for i in range(n):
        cx, cy = W / 2 + rng.uniform(-6, 6), H / 2 + rng.uniform(-6, 6)
        r = rng.uniform(0.3, 0.7) * H
        inside = np.hypot(xx - cx, yy - cy) < r
        img = np.where(inside, 130, 5) + rng.normal(0, 2, (H, W))
        if i % 3 == 2:
            img = np.full((H, W), 100.0) + rng.normal(0, 3, (H, W))
            img[:, :4] = rng.uniform(0, 30, (H, 4))
        out[i] = np.clip(np.rint(img), 0, 255).astype(np.uint8)[..., None]
    return out


# candidates 2 (h + v): up to one, two, three and four blocks of points;
# attempts around a tile, a wavefront and a workgroup; 0 lanes: the rule, which
# takes 4 lanes for one frame and 1 lane for 130 frames of 2 groups
@pytest.mark.parametrize("frames,strips,attempts,lanes", [
    (1, (4, 3), 15, 0), (1, (16, 16), 17, 0), (2, (17, 16), 64, 2), (2, (32, 32), 65, 4),
    (3, (33, 32), 129, 2), (2, (48, 48), 63, 0), (2, (64, 64), 255, 0), (130, (36, 36), 257, 0),
    (130, (9, 8), 511, 0),
])
def test_tile_edges(torch_dev, frames, strips, attempts, lanes):
    e = api.Estimator(0)
    e.set_option("schedule", "split")
    e.set_option("ransac_lanes", lanes)
    kw = dict(n_hstrips=strips[0], n_vstrips=strips[1], ransac_attempts=attempts, t_px=1)
    g, r, bits = parity._full_parity(torch_dev, e, _frames(frames, 120, 90, attempts), kw)
    assert bits[0] == bits[1]
    e.close()
