"""Solves over slices where a wave's passes change: one slice each below 4096
workgroups of four waves, then two, and a last workgroup that has few."""
import numpy as np
import pytest

from test_gpu_resident import _t, banded, check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["standard", "single"])
@pytest.mark.parametrize("n", [64 * 4 * 4088 + 1, 64 * 4 * 4095, 64 * 4 * 4095 + 1, 64 * 4 * 4096 + 65])
def test_slices_passes(cuda, n, form):
    from paper_1107_0538_amd import Solver

    a = banded(n, (1,), seed=3)
    b = np.random.default_rng(n).uniform(-1, 1, n)
    x, info = Solver(a, form=form).solve(_t(b, cuda))
    check(a, b, x.cpu().numpy(), info, form)


@pytest.mark.parametrize("n,longest", [(40001, 1), (40064, 2), (40063, 63), (40127, 64)])
def test_slices_are_filled(cuda, n, longest):
    # Rows of the longest length and a few short of it, the last slice ragged: up to the 64
    # entries that a slice takes, in no order of columns.  The product is the oracle's bits.
    import oracle
    import workloads as W
    from paper_1107_0538_amd import Solver, capi

    rng = np.random.default_rng(longest)
    cnt = longest - (rng.random(n) < 0.3) * rng.integers(0, longest // 3 + 1, n)
    cnt[-1] = longest
    rowptr = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
    rows = np.repeat(np.arange(n), cnt)
    col = np.clip(rows + rng.integers(-30000, 30000, len(rows)), 0, n - 1).astype(np.int32)
    a = W.CSR(n, rowptr, col, rng.uniform(-1, 1, len(rows)))
    x = rng.uniform(-1, 1, n)
    s = Solver(a, precond="none")
    assert s.config()["kernels"] >> 8 == capi.CG_KERNELS_SLICES
    assert np.array_equal(s.spmv(_t(x, cuda)).cpu().numpy(), oracle.spmv(a, x))
