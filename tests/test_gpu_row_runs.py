"""Multi-column products that take four rows together, at the edges of what they take.

Four rows whose entries are runs of three, each row's one column after the
row's before, share the rows of X that they read; every other four are walked
row by row.  Matrices with both kinds next to each other: every column of spmm
is bitwise the oracle's sequential product, and infinities and NaN reach only
the rows that refer to them.
"""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


def _t(a, dev):
    import torch

    return torch.as_tensor(np.ascontiguousarray(a), device=dev)


def runs(n, starts, seed, spoil):
    """Row i holds the runs i + o, i + o + 1, i + o + 2 for o in starts, as far as they fit; every
    spoil-th row reversed, shortened or lengthened by a column."""
    rng = np.random.default_rng(seed)
    rows = []
    for i in range(n):
        c = [i + o + j for o in starts for j in range(3) if 0 <= i + o and i + o + 2 < n]
        if spoil and i % spoil == 0:
            kind = (i // spoil) % 3
            c = c[::-1] if kind == 0 else c[:-1] if kind == 1 else c + [int(rng.integers(0, n))]
        rows.append(c)
    rowptr = np.concatenate([[0], np.cumsum([len(c) for c in rows])]).astype(np.int32)
    col = np.array([c for r in rows for c in r], dtype=np.int32)
    return W.CSR(n, rowptr, col, rng.uniform(-1, 1, col.size))


@pytest.mark.parametrize("s", [1, 2, 3, 31, 32, 33, 63, 64])
@pytest.mark.parametrize("n,starts,spoil", [
    (5, (-1,), 0), (8, (0,), 0), (97, (-1,), 0),                                       # one run: 3 entries
    (130, (-20, -1, 17), 13), (131, (-20, -9, -1, 17), 0),                             # 9 and 12: a full step, and one over
    (1000, tuple(range(-60, 60, 13)), 29), (1003, tuple(range(0, 33, 3)), 0),          # 30 and 33 entries
])
def test_spmm_runs_bitwise(cuda, n, starts, spoil, s):
    from paper_1107_0538_amd import Solver

    a = runs(n, starts, n, spoil)
    X = np.random.default_rng(s).uniform(-1, 1, (n, s))
    X[n // 2, 0], X[n // 3, s - 1], X[n - 1, s // 2] = np.inf, np.nan, -np.inf
    Y = Solver(a, precond="none").spmm(_t(X, cuda)).cpu().numpy()
    for j in range(s):
        assert np.array_equal(Y[:, j], oracle.spmv(a, X[:, j]), equal_nan=True), j


@pytest.mark.parametrize("s", [1, 2, 5, 33, 64])
def test_multi_columns_stop_apart(cuda, s):
    # Columns that stop at different iterations, one that starts solved and one with b = 0: what an
    # iteration leaves to the next is done for each.
    from paper_1107_0538_amd import Solver

    a, _ = W.problem(9, 4)[:2]
    rng = np.random.default_rng(s)
    x0 = rng.uniform(-1, 1, (a.n, s))
    B = np.stack([oracle.spmv(a, rng.uniform(-1, 1, a.n) * 10.0 ** -(j % 4)) for j in range(s)], 1)
    for j in range(0, s, 3):
        exact = rng.uniform(-1, 1, a.n)
        B[:, j] = oracle.spmv(a, exact)
        x0[:, j] = exact + (1e-6 * rng.uniform(-1, 1, a.n) if j % 2 else 0.0)
    if s > 1:
        B[:, 1] = 0.0
    solver = Solver(a)
    X, infos = solver.solve_multi(_t(B, cuda), X0=_t(x0, cuda), tol=1e-10)
    X = X.cpu().numpy()
    for j in range(s):
        x, info = solver.solve(_t(B[:, j], cuda), x0=_t(x0[:, j], cuda), tol=1e-10)
        assert abs(infos[j]["iters"] - info["iters"]) <= 2
        assert infos[j]["relres_true"] <= 1e-10
        x = x.cpu().numpy()
        assert np.linalg.norm(X[:, j] - x) <= 1e-8 * max(np.linalg.norm(x), 1.0), j
