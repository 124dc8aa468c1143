"""Half strips that several workgroups share: frames whose half strips are longer
than a workgroup's share of the steps (a lone frame; one with two strips), or end
anywhere in it, give the candidates that they have in a batch of many, on every
call of a plan (the words that workgroups meet in are left as they were)."""
import numpy as np
import pytest

from paper_2210_14771_amd import api, train_scorer

from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def est():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    e = api.Estimator(0)
    e.set_model(train_scorer.load_model())
    e.set_model_2d(train_scorer.load_model_2d())
    yield e
    e.close()


@pytest.mark.parametrize("scorer", [1, 2])
@pytest.mark.parametrize("w,h,n_h,n_v", [(4096, 64, 1, 0), (64, 4096, 0, 1), (1920, 1080, 1, 1),
                                         (1623, 882, 8, 15), (2142, 1416, 32, 8)])
def test_shared_half_strips(est, w, h, n_h, n_v, scorer):
    import torch
    rng = np.random.default_rng(w + h)
    frames = torch.from_numpy(rng.integers(0, 256, (3, h, w, 3), dtype=np.uint8)).cuda()
    p = api.default_params(n_hstrips=n_h, n_vstrips=n_v, ransac_attempts=64, scorer=scorer)
    say(f"strip shares, scorer {scorer}, {w}x{h}, {n_h} + {n_v}")
    _, pts = est.debug_candidates([frames[f % 3] for f in range(120)], p, list(range(120)))
    torch.cuda.synchronize()
    many = pts.cpu().numpy()
    for f in range(3, 120):
        np.testing.assert_array_equal(many[f], many[f % 3])
    for n in (1, 2, 3, 7):
        batch = [frames[f % 3] for f in range(n)]
        for call in range(3):
            _, pts = est.debug_candidates(batch, p, list(range(n)))
            torch.cuda.synchronize()
            np.testing.assert_array_equal(pts.cpu().numpy(), many[:n])
    # sub-batches on two streams, each with words of its own
    est.set_option("pipeline", 4)
    try:
        for call in range(3):
            _, pts = est.debug_candidates([frames[f % 3] for f in range(9)], p, list(range(9)))
            torch.cuda.synchronize()
            np.testing.assert_array_equal(pts.cpu().numpy(), many[:9])
    finally:
        est.set_option("pipeline", 0)
