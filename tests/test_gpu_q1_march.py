"""The operator's product marching along z: every split of lines over lanes and of planes over
workgroups is bitwise the sequential product of the assembled matrix, also with infinities and NaN
among the values and coefficients, and with an infinite mass term (which the general kernel takes)."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("n,c", [(49, 1e-3), (50, 1e-3), (51, 0.0), (60, np.inf), (63, 1.0), (64, 1e-3), (65, 1e-3), (128, 1e-3),
                                 (129, 1e-3), (131, 1e-3)])
def test_q1_march_bitwise(cuda, n, c, odd):
    import torch

    from paper_1107_0538_amd import q1_apply, q1_assemble

    rng = np.random.default_rng(n)
    sig = np.exp(rng.standard_normal((n - 1,) * 3))
    x = rng.standard_normal(n ** 3)
    if odd:
        x[[0, n - 1, n * n // 2, n ** 3 // 2, n ** 3 - 1]] = [np.inf, np.nan, -np.inf, -0.0, np.inf]
        sig.flat[[0, sig.size // 2, sig.size - 1]] = [np.inf, np.nan, np.inf]
    st, xt = torch.as_tensor(sig, device=cuda), torch.as_tensor(x, device=cuda)
    y = q1_apply(n, st, xt, c=c).cpu().numpy()
    m = q1_assemble(n, st, c=c)
    host = W.CSR(m.n, m.rowptr.cpu().numpy(), m.col.cpu().numpy(), m.val.cpu().numpy())
    assert np.array_equal(y, oracle.spmv(host, x), equal_nan=True)
