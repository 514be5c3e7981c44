"""A forward pass takes a launch per layer for small networks and batches, else
large tiles: rows of a batch on either side of the line hold the same bits, as
both add a row's products in one order."""
import numpy as np
import pytest

from test_gpu_learned import _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("dims,batches", [
    ([24, 64, 64, 64], (14080, 14144, 16384, 16385)),  # 220, 221, 256 and 257 tiles of 64
    ([512, 512, 512], (1728, 1792, 2048)),             # 216, 224, 256
])
def test_forward_on_both_sides(cuda, dims, batches, precision):
    from paper_1107_0538_amd import learned

    rng = np.random.default_rng(len(dims))
    flat = np.concatenate([np.concatenate([rng.uniform(-1, 1, a * b) * np.sqrt(1.5 / a), rng.uniform(-0.5, 0.5, b)])
                           for a, b in zip(dims, dims[1:])]).astype(np.float32)
    net = learned.MLP(dims, precision, max_batch=max(batches))
    net.set_params(flat)
    X = _t(rng.uniform(-1, 1, (max(batches), dims[0])).astype(np.float32), cuda)
    few = net.forward(X[:64].contiguous())
    for batch in batches:
        Y = net.forward(X[:batch].contiguous())
        assert (Y[:64] == few).all() and (Y[-1] == net.forward(X[batch - 1:batch].contiguous())[0]).all(), batch
