"""Learned candidates at the edges of a wave's steps: half strips shorter than a
step, of one step (64 positions less the halo's 16, or 6 of the 2-D network), of
one position more and of several, alone (a half strip shared by several waves),
in batches that leave fewer waves to a half strip, and among frames of other
shapes."""
import numpy as np
import pytest

from oracle import cnn, cnn2d
from paper_2210_14771_amd import api, synth

import test_gpu_cnn2d as two_d
from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# frame sizes: halves of 8; 48 and 49; 56 and 57 (the second has a longer
# second half); 58 and 59; 112 and 113; 160 and 119
@pytest.mark.parametrize("scorer", [1, 2])
@pytest.mark.parametrize("w,h", [(16, 16), (96, 99), (113, 112), (116, 119), (225, 227),
                                 (321, 239)])
def test_candidates_at_step_edges(torch_dev, w, h, scorer):
    torch = torch_dev
    rng = np.random.default_rng(w)
    est = api.Estimator(0)
    if scorer == 1:
        net = cnn
        params = [(m, b + rng.normal(0, 0.1, b.shape)) for m, b in cnn.init_params(7)]
        est.set_model(cnn.flat_params(params))
    else:
        net = cnn2d
        params = two_d._params(7)
        est.set_model_2d(cnn2d.flat_params(params))
    frame, _ = synth.make_frame(synth.SMALL_640x480, 3, w, h)
    # a crop whose rows start at any alignment and end before the buffer's
    big = torch.from_numpy(rng.integers(0, 256, (h + 3, w + 5, 3), dtype=np.uint8)).cuda()
    big[1:h + 1, 3:w + 3] = torch.from_numpy(frame).cuda()
    views = {"whole": torch.from_numpy(frame).cuda(), "crop": big[1:h + 1, 3:w + 3]}
    p = api.default_params(n_hstrips=4, n_vstrips=3, ransac_attempts=64, scorer=scorer)
    halves = net.learned_half_strip_scores(frame, params, 4, 3)
    tol = 0.01   # as for the candidates of larger frames
    alone = None
    for name, view in views.items():
        for n in (1, 20, 40, 160):
            say(f"learned steps, scorer {scorer}, {w}x{h} {name} x {n}")
            _, pts = est.debug_candidates([view] * n, p, list(range(n)))
            torch.cuda.synchronize()
            g = api.points_numpy(pts)
            if alone is None:
                alone = g[0].copy()
                for c, (xs, ys, sc) in enumerate(halves):
                    at = np.flatnonzero((xs == alone[c]["x"]) & (ys == alone[c]["y"]))
                    assert at.size == 1, (c, alone[c])
                    assert sc[at[0]] >= sc.max() - tol, (c, sc[at[0]], sc.max())
                    assert abs(float(alone[c]["score"]) - sc[at[0]]) <= tol
            for f in range(n):
                assert np.array_equal(g[f], alone), (name, n, f)
    # every third of a batch of several shapes
    other = [torch.from_numpy(rng.integers(0, 256, (hh, ww, 3), dtype=np.uint8)).cuda()
             for ww, hh in ((64, 48), (640, 480))]
    for n in (3, 39, 240):
        say(f"learned steps, scorer {scorer}, {w}x{h} mixed x {n}")
        batch = [views["crop"] if f % 3 == 1 else other[f % 3 // 2] for f in range(n)]
        _, pts = est.debug_candidates(batch, p, list(range(n)))
        torch.cuda.synchronize()
        g = api.points_numpy(pts)
        for f in range(1, n, 3):
            assert np.array_equal(g[f], alone), ("mixed", n, f)
