"""Targets and weights of positions that carry no loss (outside a window's strip
range) are not read into the gradients or the loss: with values there that are
not numbers, both equal, bit for bit, those with zeros there."""
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


# ranges that begin after the first output (position 8), end before the last
# (119), do both, or hold no position at all
@pytest.mark.parametrize("net", ["1d", "2d"])
@pytest.mark.parametrize("lo,hi", [(9, 128), (0, 119), (40, 77), (64, 64), (120, 128)])
def test_values_without_loss_do_not_matter(torch_dev, lo, hi, net):
    torch = torch_dev
    rng = np.random.default_rng(lo + hi)
    n = 5
    e = api.Estimator(0)
    win, geom, ranges = two_d._windows(rng, n)
    ranges[1::2] = (lo, hi)
    if net == "1d":
        e.set_model(cnn.flat_params(one_d._spread_params(3)))
        args, gradients = (win, ranges), e.cnn_gradients
    else:
        e.set_model_2d(cnn2d.flat_params(two_d._params(3)))
        args, gradients = (win, geom, ranges), e.cnn2d_gradients
    pos = np.arange(8, 120)
    used = (pos >= ranges[:, :1]) & (pos < ranges[:, 1:])
    targets = rng.uniform(0, 1, (n, 112)).astype(np.float32)
    weights = rng.uniform(0, 1, (n, 112)).astype(np.float32)
    out = []
    for fill in (0.0, np.nan, np.inf):
        say(f"no-loss positions, {net}, range {lo}..{hi}, fill {fill}")
        t, w = np.where(used, targets, np.float32(fill)), np.where(used, weights, np.float32(fill))
        grad, loss = gradients(*two_d._dev(torch, *args, t, w), 1.0 / n)
        torch.cuda.synchronize()
        out.append((grad.cpu().numpy(), loss.cpu().numpy()))
    assert np.isfinite(out[0][0]).all() and np.isfinite(out[0][1]).all()
    for got in out[1:]:
        np.testing.assert_array_equal(got[0], out[0][0])
        np.testing.assert_array_equal(got[1], out[0][1])
    e.close()
