"""Window batches at their edges, for both learned scorers: gradients of one
window (one partial vector) and of counts on both sides of a sweep of the
column sums (64 rows) and of a workgroup's share; logits at counts around the
launch's workgroups."""
import numpy as np
import pytest

from oracle import cnn, cnn2d
from paper_2210_14771_amd import api

import test_gpu_cnn as one_d
import test_gpu_cnn2d as two_d
from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _check(g, ref, slices, max_rel, norm_rel):
    for name, sl in slices:
        d = g[sl] - ref[sl]
        scale = np.abs(ref[sl]).max()
        assert np.abs(d).max() <= max_rel * scale, (name, np.abs(d).max(), scale)
        assert np.linalg.norm(d) <= norm_rel * np.linalg.norm(ref[sl]), name


# A window alone averages over 112 positions instead of thousands: a signal
# whose bfloat16 rounding falls the other way (2^-8 of one of 112 terms) may
# move a tensor's entries by more than in the tests of many windows; twice
# their bounds.
SMALL = 2.0


@pytest.mark.parametrize("n", [1, 2, 63, 65, 129])
def test_gradients_of_few_windows(torch_dev, n):
    torch = torch_dev
    say(f"gradients of {n} windows")
    e = api.Estimator(0)
    rng = np.random.default_rng(40 + n)
    params = one_d._spread_params(7)
    e.set_model(cnn.flat_params(params))
    case = one_d._train_case(rng, n)
    scale = float(np.float32(1.0 / max(case[3].sum(), 1.0)))
    grad, loss = e.cnn_gradients(*two_d._dev(torch, *case), scale)
    torch.cuda.synchronize()
    ref_loss, ref = one_d._oracle_window_grads(*case, params, scale)
    assert abs(loss.item() - ref_loss) <= one_d.LOSS_REL * abs(ref_loss)
    _check(grad.cpu().numpy().astype(np.float64), ref, one_d._param_slices(),
           SMALL * one_d.GRAD_MAX_REL, SMALL * one_d.GRAD_NORM_REL)

    params = two_d._params(17)
    e.set_model_2d(cnn2d.flat_params(params))
    case = two_d._case(rng, n)
    scale = float(np.float32(1.0 / max(case[4].sum(), 1.0)))
    grad, loss = e.cnn2d_gradients(*two_d._dev(torch, *case), scale)
    torch.cuda.synchronize()
    ref_loss, ref = cnn2d.loss_and_grads(*case, params, scale, grad_bf16=True)
    assert abs(loss.item() - ref_loss) <= two_d.LOSS_REL * abs(ref_loss)
    g = grad.cpu().numpy().astype(np.float64)
    assert np.all(g[:cnn2d.N_NORM] == 0)
    _check(g, ref, two_d._slices(), SMALL * two_d.GRAD_MAX_REL, SMALL * two_d.GRAD_NORM_REL)
    e.close()


# 1024 workgroups of one window (2-D) or two (1-D): counts around both, and
# windows of both orientations changing places at every share
@pytest.mark.parametrize("n", [1, 3, 1025, 2051])
def test_logits_do_not_depend_on_the_batch(torch_dev, n):
    torch = torch_dev
    say(f"logits of {n} windows")
    e = api.Estimator(0)
    rng = np.random.default_rng(n)
    params1, params2 = one_d._spread_params(8), two_d._params(18)
    e.set_model(cnn.flat_params(params1))
    e.set_model_2d(cnn2d.flat_params(params2))
    win, geom, ranges = two_d._windows(rng, n)
    dw, dg, dr = two_d._dev(torch, win, geom, ranges)
    z1, z2 = e.cnn_window_logits(dw, dr), e.cnn2d_window_logits(dw, dg, dr)
    some = sorted({0, n - 1, n // 2, *rng.integers(0, n, 5).tolist()})
    for i in some:
        one = slice(i, i + 1)
        assert torch.equal(e.cnn_window_logits(dw[one], dr[one]), z1[one])
        assert torch.equal(e.cnn2d_window_logits(dw[one], dg[one], dr[one]), z2[one])
    for i in some[:3]:
        lo, hi = int(ranges[i, 0]), int(ranges[i, 1])
        w1 = [(cnn.bf16(w), b) for w, b in cnn.unflat_params(cnn.flat_params(params1))]
        for z, ref in ((z1, cnn.window_forward(win[i], lo, hi, w1)),
                       (z2, cnn2d.window_forward(win[i], geom[i], lo, hi, params2))):
            ok = ~np.isnan(ref)
            assert np.abs(z[i].cpu().numpy()[ok] - ref[ok]).max() <= two_d.LOGIT_TOL
    e.close()
