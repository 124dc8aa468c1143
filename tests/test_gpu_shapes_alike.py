"""Batches of several shapes through every route: the entry point without
allocation gives the results of the cached plans bit for bit, with each scorer,
where shapes repeat out of order, share one area, or fill whole frames per XCD."""
import numpy as np
import pytest

from paper_2210_14771_amd import api, train_scorer

from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.fixture(scope="module")
def est(torch_dev):
    e = api.Estimator(0)
    e.set_model(train_scorer.load_model())
    e.set_model_2d(train_scorer.load_model_2d())
    yield e
    e.close()


SIZES = {"few": [(320, 240), (641, 479), (64, 48), (320, 240), (1280, 720)],
         "one area": [(640, 480), (480, 640)] * 5,
         "many": [(320, 240), (641, 479), (64, 48), (400, 300)] * 12}


@pytest.mark.parametrize("scorer", [0, 1, 2])
@pytest.mark.parametrize("name", sorted(SIZES))
def test_routes_agree_on_several_shapes(torch_dev, est, name, scorer):
    torch = torch_dev
    say(f"shapes alike: {name}, scorer {scorer}")
    rng = np.random.default_rng(5)
    views = [torch.from_numpy(rng.integers(0, 256, (h, w, 3), dtype=np.uint8)).cuda()
             for w, h in SIZES[name]]
    p = api.default_params(n_hstrips=5, n_vstrips=6, ransac_attempts=200, scorer=scorer,
                           fallback_inlier_frac=0.5 if scorer else 0.0)
    a, b = est.estimate_area(views, p), est.estimate_area_noalloc(views, p)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(a.raw.cpu().numpy(), b.raw.cpu().numpy())
    # each frame as it comes out of a batch of its own shape
    _, pts = est.debug_candidates(views, p)
    for shape in sorted(set(SIZES[name])):
        idx = [i for i, s in enumerate(SIZES[name]) if s == shape]
        _, own = est.debug_candidates(torch.stack([views[i] for i in idx]), p, idx)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(pts[idx].cpu().numpy(), own.cpu().numpy())
