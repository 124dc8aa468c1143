"""An SGD step writes every weight's copies in the device model: logits and
gradients after two steps equal, bit for bit, those of a context that loads the
updated weights (both orientations of the 2-D network)."""
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


@pytest.mark.parametrize("net", ["1d", "2d"])
def test_step_updates_every_copy(torch_dev, net):
    torch = torch_dev
    rng = np.random.default_rng(11)
    n = 40
    if net == "1d":
        p0 = cnn.flat_params(one_d._spread_params(3)).astype(np.float32)
        win, ranges, targets, weights = one_d._train_case(rng, n)
        args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (win, ranges)]
    else:
        p0 = cnn2d.flat_params(two_d._params(3)).astype(np.float32)
        win, geom, ranges = two_d._windows(rng, n)
        targets = rng.uniform(0, 1, (n, 112)).astype(np.float32)
        weights = rng.uniform(0, 1, (n, 112)).astype(np.float32)
        args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (win, geom, ranges)]
        assert set(geom[:, 0]) == {0, 1}
    loss_args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (targets, weights)]

    def load(e, p):
        (e.set_model if net == "1d" else e.set_model_2d)(p)

    def outputs(e):
        if net == "1d":
            z = e.cnn_window_logits(*args)
            g, loss = e.cnn_gradients(*args, *loss_args, 1.0 / n)
        else:
            z = e.cnn2d_window_logits(*args)
            g, loss = e.cnn2d_gradients(*args, *loss_args, 1.0 / n)
        torch.cuda.synchronize()
        return z.cpu().numpy(), g.cpu().numpy(), loss.cpu().numpy()

    say(f"update of every copy, {net}")
    a = api.Estimator(0)
    load(a, p0)
    for _ in range(2):
        g = torch.from_numpy((rng.standard_normal(p0.size) * 0.01).astype(np.float32)).cuda()
        (a.cnn_sgd_step if net == "1d" else a.cnn2d_sgd_step)(g, 0.5, 0.9)
    torch.cuda.synchronize()
    p = a.get_model() if net == "1d" else a.get_model_2d()
    assert not np.array_equal(p, p0)
    b = api.Estimator(0)
    load(b, p)
    for x, y in zip(outputs(a), outputs(b)):
        np.testing.assert_array_equal(x, y)
