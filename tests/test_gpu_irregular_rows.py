"""Multi-column products and solves on rows that are not runs.

Which kernel takes a matrix is a matter of its rows: a row per wave for small
matrices, else four rows at a time, where fours of unequal or long rows are
walked as a stream of entries (64 of them through LDS at a time, 8 gathered
together) if there are more than a few of them.  Matrices on both sides of the
lines: every column of spmm is bitwise the oracle's sequential product, and
infinities and NaN reach only the rows that refer to them; solves meet the
single-system criteria.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from conftest import tol_recomputed
from test_gpu_row_runs import runs

pytestmark = pytest.mark.gpu


def _t(a, dev):
    import torch

    return torch.as_tensor(np.ascontiguousarray(a), device=dev)


def rows_of(lengths, seed):
    """A matrix with rows of these lengths, columns at random (unsorted, some twice)."""
    rng = np.random.default_rng(seed)
    n = len(lengths)
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    return W.CSR(n, rowptr, rng.integers(0, n, rowptr[-1]).astype(np.int32), rng.uniform(-1, 1, rowptr[-1]))


def unequal(n, most, seed):
    rng = np.random.default_rng(seed)
    k = rng.integers(0, most + 1, n)
    k[n // 3:n // 3 + 9] = 0
    return k


CASES = {
    "one length, a row per wave": lambda: rows_of([27] * 16384, 1),
    "one length, fours": lambda: rows_of([27] * 16385, 2),
    "one length, the longest side by side": lambda: rows_of([32] * 16387, 3),
    "runs, a row per wave": lambda: runs(6144, (-60, -1, 40), 4, 0),
    "runs, fours": lambda: runs(6145, (-60, -1, 40), 5, 0),
    "runs, one each": lambda: runs(6146, (-1,), 15, 0),
    "runs, a step and one over": lambda: runs(6147, (-20, -9, -1, 17), 16, 13),
    "runs, longer than half a wave": lambda: runs(16391, tuple(range(0, 33, 3)), 17, 0),
    "runs, some spoilt": lambda: runs(6147, tuple(range(-60, 60, 13)), 6, 29),
    "a few unequal fours side by side": lambda: rows_of([24, 20, 3, 24] + [24] * 16410, 7),
    "unequal, a row per wave": lambda: rows_of(unequal(4001, 40, 8), 9),
    "unequal, streams": lambda: rows_of(unequal(16386, 24, 10), 11),
    "long, parts of 64": lambda: rows_of(
        [2] * 16384 + [63, 1, 0, 0, 64, 0, 0, 0, 32, 32, 1, 0, 60, 60, 60, 60, 128, 129, 33, 7], 12),
    "one long row": lambda: rows_of([3] * 8500 + [3000] + [3] * 8502, 13),
    "no entries": lambda: rows_of([0] * 16397 + [40] + [0] * 3, 14),
}


@pytest.mark.parametrize("s", [1, 2, 3, 33, 64])
@pytest.mark.parametrize("case", list(CASES))
def test_spmm_irregular_bitwise(cuda, case, s):
    from paper_1107_0538_amd import Solver

    a = CASES[case]()
    X = np.random.default_rng(s).uniform(-1, 1, (a.n, s))
    X[a.n // 2, 0], X[a.n // 3, s - 1], X[a.n - 1, s // 2] = np.inf, np.nan, -np.inf
    Y = Solver(a, precond="none").spmm(_t(X, cuda)).cpu().numpy()
    for j in range(s):
        assert np.array_equal(Y[:, j], oracle.spmv(a, X[:, j]), equal_nan=True), j


SURPLUS = 0.05


def spd(lengths, seed):
    """Symmetric, with about these many links per row and a diagonal that exceeds the row's other
    entries by SURPLUS, so that no eigenvalue is below that."""
    import scipy.sparse as sp

    rng = np.random.default_rng(seed)
    i = np.repeat(np.arange(len(lengths)), lengths)
    j = rng.integers(0, len(lengths), i.size)
    w = -rng.uniform(0.1, 1.0, i.size)
    m = sp.coo_matrix((w, (i, j)), shape=(len(lengths),) * 2).tocsr()
    m = m + m.T
    m.setdiag(0.0)
    m = (m + sp.diags(np.asarray(abs(m).sum(1)).ravel() + SURPLUS)).tocsr()
    m.eliminate_zeros()
    m.sort_indices()
    return W.CSR(m.shape[0], m.indptr.astype(np.int32), m.indices.astype(np.int32), m.data.astype(np.float64))


@pytest.mark.parametrize("s", [1, 5, 64])
@pytest.mark.parametrize("most", [3, 30])
def test_multi_column_solves_irregular(cuda, most, s):
    from paper_1107_0538_amd import Solver

    a = spd(unequal(3001, most, most), most)
    B = np.random.default_rng(s).uniform(-1, 1, (a.n, s))
    solver = Solver(a, fp32_copy=True)
    alone = [oracle.pcg(a, B[:, j]) for j in range(min(s, 4))]
    for name in ("solve_multi", "solve_block", "solve_multi_mixed"):
        X, infos = getattr(solver, name)(_t(B, cuda))
        X = X.cpu().numpy()
        assert all(i["status"] == 0 for i in infos)
        assert all(oracle.relres(a, B[:, j], X[:, j]) <= tol_recomputed(a.n) for j in range(s)), name
        for j, (xo, io) in enumerate(alone):
            # Two residuals within the tolerance: A (x - xo) = ro - r.
            assert np.linalg.norm(X[:, j] - xo) <= 2 * tol_recomputed(a.n) * np.linalg.norm(B[:, j]) / SURPLUS
            if name == "solve_multi":
                assert abs(infos[j]["iters"] - io["iters"]) <= 2
