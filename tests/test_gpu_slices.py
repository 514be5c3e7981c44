"""Products and solves over slices of 64 rows, at the edges of what they take.

Slices serve spmv, and solves of systems that the on-chip solver does not
hold, where neighbouring rows are about equally long (the padding of a slice to
its longest row costs at most a quarter), no row has more than 64 entries and
every column lies within 32 Ki of its slice's first row.  Matrices on both
sides of each line: spmv is bitwise the oracle's sequential product, solves
meet the single-system criteria.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_resident import banded, check

pytestmark = pytest.mark.gpu


def _t(a, dev):
    import torch

    return torch.as_tensor(np.ascontiguousarray(a), device=dev)


@pytest.mark.parametrize("n,offsets", [
    (1, ()), (63, (1, 5)), (64, (1, 5)), (65, (1, 5)), (1000, ()),          # one slice, two, ragged, 1 entry a row
    (5000, tuple(range(1, 7))), (5000, tuple(range(1, 8))),                  # 13 and 15 entries: one chunk and two
    (5000, tuple(range(1, 14))), (5000, tuple(range(1, 15))),                # 27 and 29
    (3000, tuple(range(1, 32))), (3000, tuple(range(1, 33))),                # 63 and 65 entries: slices and tiles
    (70000, (1, 32704)), (70000, (1, 32705)), (70000, (1, 32767)), (70000, (1, 33000)),  # the farthest column
    (3000, (2000,)),                                                         # half the rows have a second entry
])
def test_slices_product_bitwise(cuda, n, offsets):
    from paper_1107_0538_amd import Solver

    a = banded(n, offsets, seed=n, shuffle=n <= 1000)
    x = np.random.default_rng(n).uniform(-1, 1, n)
    s = Solver(a)
    assert np.array_equal(s.spmv(_t(x, cuda)).cpu().numpy(), oracle.spmv(a, x))


@pytest.mark.parametrize("n,offsets", [
    (39999, (1, 5)), (40000, (1, 5)), (40001, ()), (40033, tuple(range(1, 7))), (40063, tuple(range(1, 8))),  # tiles, then slices
    (40064, tuple(range(1, 14))), (40065, tuple(range(1, 15))), (41000, tuple(range(1, 32))), (41000, tuple(range(1, 33))),
])
def test_slices_product_from_its_smallest_size(cuda, n, offsets):
    from paper_1107_0538_amd import Solver

    a = banded(n, offsets, seed=n)
    x = np.random.default_rng(n).uniform(-1, 1, n)
    x[[5, n // 2, n - 1]] = [np.inf, -np.inf, np.nan]
    y = Solver(a).spmv(_t(x, cuda)).cpu().numpy()
    assert np.array_equal(y, oracle.spmv(a, x), equal_nan=True)


def test_slices_product_rows_without_entries_and_infinities(cuda):
    # Empty rows sum to zero, and an infinity reaches only the rows that refer to it.
    from paper_1107_0538_amd import Solver

    rng = np.random.default_rng(3)
    n = 300
    cnt = rng.integers(0, 3, n)
    cnt[64:128] = 0  # a whole slice
    cnt[-40:] = 0
    rowptr = np.concatenate([[0], np.cumsum(np.maximum(cnt, 0))]).astype(np.int32)
    col = rng.integers(0, n, rowptr[-1]).astype(np.int32)
    a = W.CSR(n, rowptr, col, rng.uniform(-1, 1, rowptr[-1]))
    x = rng.uniform(-1, 1, n)
    x[[5, 70, 299]] = [np.inf, -np.inf, np.nan]
    y = Solver(a, precond="none").spmv(_t(x, cuda)).cpu().numpy()
    assert np.array_equal(y, oracle.spmv(a, x), equal_nan=True)


@pytest.mark.parametrize("values", ["fp64", "fp32"])
@pytest.mark.parametrize("n,offsets", [(262145, (1, 600)), (300001, (1, 30, 900)), (6000, tuple(range(1, 16)))])
def test_slices_solve(cuda, n, offsets, values):
    from paper_1107_0538_amd import Solver

    a = banded(n, offsets, seed=n)
    b = np.random.default_rng(n + 1).uniform(-1, 1, n)
    s = Solver(a, fp32_copy=values == "fp32", history=values == "fp64")
    solve = s.solve if values == "fp64" else s.solve_mixed_matrix
    x, info = solve(_t(b, cuda))
    check(a, b, x.cpu().numpy(), info, "standard")
    if values == "fp64":
        _, _, ho = oracle.pcg(a, b, history=True)
        assert np.allclose(s.history()[:10], ho[:10], rtol=1e-8)
    # A start vector, the limit at both parities, b = 0, NaN, and clean again.
    x0 = np.random.default_rng(2).uniform(-1, 1, n)
    for maxit in (1, 2, 3):
        x, info = solve(_t(b, cuda), x0=_t(x0, cuda), maxit=maxit)
        assert info["status"] == 1 and info["iters"] == maxit
        if values == "fp64":
            xo, io = oracle.pcg(a, b, x0=x0, maxit=maxit)
            assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-9 * np.linalg.norm(xo)
            assert abs(info["relres_true"] - io["relres_true"]) <= 1e-8 * io["relres_true"]
    x, info = solve(_t(np.zeros(n), cuda), x0=_t(x0, cuda))
    assert info["status"] == 0 and info["iters"] == 0 and not bool(x.any())
    bn = b.copy()
    bn[7] = np.nan
    assert solve(_t(bn, cuda))[1]["status"] == 2
    x, info = solve(_t(b, cuda))
    check(a, b, x.cpu().numpy(), info, "standard")


def test_slices_solve_breakdown(cuda):
    # An indefinite matrix of rows too long for the on-chip solver: p'Ap <= 0
    # at the first iterations, where x's last update is already done.
    from paper_1107_0538_amd import Solver

    a = banded(4000, tuple(range(1, 16)), seed=1)
    diag = a.col == np.repeat(np.arange(a.n), np.diff(a.rowptr))
    a.val[diag & (a.col % 5 == 0)] *= -0.5
    b = np.random.default_rng(4).uniform(-1, 1, a.n)
    x, info = Solver(a, precond="none").solve(_t(b, cuda))
    xo, io = oracle.pcg(a, b, precond="none")
    assert info["status"] == io["status"] == 2 and info["iters"] == io["iters"]
    assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-9 * max(np.linalg.norm(xo), 1e-300)


@pytest.mark.parametrize("history", [False, True])
@pytest.mark.parametrize("n,offsets", [(262145, (1, 600)), (300001, (1, 30, 900)), (6000, tuple(range(1, 16)))])
def test_slices_single_reduction(cuda, n, offsets, history):
    # The single-reduction form over slices: converged, stopped by the limit, by b = 0 and at once by
    # x0, and resumed after replacements (the last one asks for more than is attainable).
    from paper_1107_0538_amd import Solver

    a = banded(n, offsets, seed=n)
    b = np.random.default_rng(n + 1).uniform(-1, 1, n)
    s = Solver(a, form="single", history=history)
    x, info = s.solve(_t(b, cuda))
    check(a, b, x.cpu().numpy(), info, "single")
    if history:
        h = s.history()
        assert h.size == info["iters"] + 1 and h[-1] <= 1e-10 < h[-2]
    x3, i3 = s.solve(_t(b, cuda), maxit=3)
    xo, io = oracle.pcg(a, b, maxit=3)
    assert i3["status"] == io["status"] == 1 and i3["iters"] == 3
    assert np.linalg.norm(x3.cpu().numpy() - xo) <= 1e-9 * np.linalg.norm(xo)
    x0, i0 = s.solve(_t(np.zeros(n), cuda), x0=x)
    assert i0["status"] == 0 and i0["iters"] == 0 and not x0.cpu().numpy().any()
    again, ia = s.solve(_t(b, cuda), x0=x, tol=1e-9)
    assert ia["status"] == 0 and ia["iters"] == 0 and (again == x).all()
    _, ir = s.solve(_t(b, cuda), tol=1e-17, maxit=2 * info["iters"] + 40)
    assert ir["status"] in (1, 2) and ir["replacements"] >= (0 if ir["status"] == 2 else 1)
    assert ir["relres_true"] <= 1e-12
