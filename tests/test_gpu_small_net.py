"""Networks that run in one launch per layer and direction, at the edges of the kernels' tiles (16
outputs, 256 terms), of the batch's chunks (128) and of the rule that chooses them (256 tiles of 64).

Forward and gradients against the FP64 oracle with the tolerances of the learned warm start's
tests (FP32 1e-5, BF16 2e-2, normwise per tensor); one training step against Adam's formula on the
gradients that the network reports, in FP64: the step is at most lr, its FP32 arithmetic a few
roundings, and the parameter is rounded once.
"""
import numpy as np
import pytest

import oracle.mlp as om
from test_gpu_learned import _t, relnorm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol", [("fp32", 1e-5), ("bf16", 2e-2)])
@pytest.mark.parametrize("dims,batch", [
    ([1, 1], 1), ([15, 17, 16], 15), ([24, 48, 48, 64], 127), ([256, 16, 257], 128), ([257, 255, 3, 5], 129),
    ([24, 256, 256, 64], 255), ([24, 100, 90, 80, 7], 257), ([24, 1024, 64], 1024), ([24, 64, 40], 16385),
])
def test_small_net(cuda, dims, batch, precision, tol):
    from paper_1107_0538_amd import learned

    rng = np.random.default_rng(batch)
    flat = np.concatenate([np.concatenate([rng.uniform(-1, 1, a * b) * np.sqrt(1.5 / a), rng.uniform(-0.5, 0.5, b)])
                           for a, b in zip(dims, dims[1:])]).astype(np.float32)
    X = rng.uniform(-1, 1, (batch, dims[0])).astype(np.float32)
    T = rng.uniform(-1, 1, (batch, dims[-1])).astype(np.float32)
    params = [(w.copy(), b.copy()) for w, b in learned.layer_views(flat.astype(np.float64), dims)]
    net = learned.MLP(dims, precision, max_batch=batch)
    net.set_params(flat)
    Yo, cache = om.forward(params, X.astype(np.float64))
    assert relnorm(net.forward(_t(X, cuda)).cpu().numpy(), Yo) <= tol
    g, loss = net.gradients(_t(X, cuda), _t(T, cuda))
    go = om.backward(params, cache, Yo, T.astype(np.float64))
    lo = om.loss(Yo, T.astype(np.float64))
    assert abs(loss - lo) <= tol * lo
    for (gw, gb), (ow, ob) in zip(learned.layer_views(g.astype(np.float64), dims), go):
        assert relnorm(gw, ow) <= tol and relnorm(gb, ob) <= tol
    assert net.train_step(_t(X, cuda), _t(T, cuda), lr=1e-3, want_loss=True) == loss
    g = g.astype(np.float64)
    step = 1e-3 * g / (np.abs(g) + 1e-8)
    p = net.get_params().astype(np.float64)
    assert np.all(np.abs(p - (flat - step)) <= 1e-3 * 1e-5 + 2.0 ** -23 * np.abs(flat))
    # The step reached the copies that the products read.
    Yn, _ = om.forward([(w.copy(), b.copy()) for w, b in learned.layer_views(p, dims)], X.astype(np.float64))
    assert relnorm(net.forward(_t(X, cuda)).cpu().numpy(), Yn) <= tol


def test_small_net_output_over_input(cuda):
    from paper_1107_0538_amd import learned

    rng = np.random.default_rng(0)
    flat = rng.uniform(-1, 1, 40 * 40 + 40).astype(np.float32)
    net = learned.MLP([40, 40], "fp32", max_batch=100)
    net.set_params(flat)
    X = _t(rng.uniform(-1, 1, (100, 40)).astype(np.float32), cuda)
    Y = net.forward(X).clone()
    assert (net.forward(X, X) == Y).all()
