"""The on-chip solver (one kernel per solve) at the edges of what it takes.

Which systems it takes is a matter of rows (one workgroup; one group of 32
workgroups up to 20480 rows; eight groups; blocks of 256, 640 or 1024
threads), of the longest row (16, 28, more: the general kernels) and of how
many foreign columns a workgroup's rows refer to.  Systems on both sides of
each line meet the single-system criteria against the CPU oracle: the same
status, +-2 iterations, the solution within 1e-8 and the recomputed true
residual within the tolerance.
"""
import threading

import numpy as np
import pytest

import oracle
import workloads as W
from conftest import mean_removed_relerr, tol_recomputed

pytestmark = pytest.mark.gpu


def _t(a, dev):
    import torch

    return torch.as_tensor(np.ascontiguousarray(a), device=dev)


def banded(n, offsets, seed=0, shuffle=False):
    """Symmetric, strictly diagonally dominant matrix with entries at the given
    offsets on both sides of the diagonal (where they exist)."""
    import scipy.sparse as sp

    rng = np.random.default_rng(seed)
    diags = {o: -rng.uniform(0.1, 1.0, n - o) for o in offsets if o < n}
    m = sp.diags([*diags.values(), *diags.values()], [*diags, *[-o for o in diags]], shape=(n, n), format="csr") \
        if diags else sp.csr_matrix((n, n))
    m = (m + sp.diags(np.asarray(abs(m).sum(axis=1)).ravel() + rng.uniform(0.05, 0.2, n))).tocsr()
    m.sort_indices()
    if shuffle:  # columns need not be sorted within a row
        for i in range(n):
            p = rng.permutation(m.indptr[i + 1] - m.indptr[i]) + m.indptr[i]
            m.indices[m.indptr[i]:m.indptr[i + 1]] = m.indices[p]
            m.data[m.indptr[i]:m.indptr[i + 1]] = m.data[p]
    return W.CSR(n, m.indptr.astype(np.int32), m.indices.astype(np.int32), m.data.astype(np.float64))


def check(a, b, x, info, form):
    xo, io = oracle.pcg(a, b, form=form)
    assert info["status"] == io["status"] == 0
    assert abs(info["iters"] - io["iters"]) <= 2, (info, io)
    assert np.linalg.norm(x - xo) <= 1e-8 * np.linalg.norm(xo)
    assert mean_removed_relerr(x, xo) <= 1e-8
    assert oracle.relres(a, b, x) <= tol_recomputed(a.n)


CASES = [
    # rows: one workgroup, two, a ragged last one, one group's limit and past it
    (1, ()), (63, (1, 7)), (64, (1, 7)), (65, (1, 7)), (1000, (1, 30)), (20480, (1, 150)), (20481, (1, 150)),
    # blocks of 256, 640 and 1024 threads over eight groups, and too many rows
    (65536, (1, 300)), (65537, (1, 300)), (163840, (1, 400)), (163841, (1, 400)), (262144, (1, 500)),
    (262145, (1, 500)),
    # longest row 16 (offsets one-sided at the ends), 17, 28, 29
    (3000, (1, 2, 3, 4, 5, 6, 7)), (3000, (1, 2, 3, 4, 5, 6, 7, 8)), (3000, tuple(range(1, 14))),
    (3000, tuple(range(1, 15))),
    # links over half the system: nearly every workgroup reads every other
    (30000, (1, 5000, 11000, 15000)), (200000, (1, 30011, 60013, 99991)),
]


@pytest.mark.parametrize("form", ["standard", "single"])
@pytest.mark.parametrize("n,offsets", CASES)
def test_resident_sizes(cuda, n, offsets, form):
    from paper_1107_0538_amd import Solver

    a = banded(n, offsets, seed=n)
    b = np.random.default_rng(n + 1).uniform(-1, 1, n)
    s = Solver(a, form=form)
    x, info = s.solve(_t(b, cuda))
    check(a, b, x.cpu().numpy(), info, form)
    x2, info2 = s.solve(_t(b, cuda))
    assert np.array_equal(x.cpu().numpy(), x2.cpu().numpy()) and info["iters"] == info2["iters"]


@pytest.mark.parametrize("form", ["standard", "single"])
def test_resident_unsorted_columns_and_start_vector(cuda, form):
    from paper_1107_0538_amd import Solver

    a = banded(2500, (1, 3, 50), seed=5, shuffle=True)
    rng = np.random.default_rng(6)
    b, x0 = rng.uniform(-1, 1, a.n), rng.uniform(-1, 1, a.n)
    x, info = Solver(a, form=form).solve(_t(b, cuda), x0=_t(x0, cuda))
    xo, io = oracle.pcg(a, b, x0=x0, form=form)
    assert info["status"] == io["status"] == 0 and abs(info["iters"] - io["iters"]) <= 2
    assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-8 * np.linalg.norm(xo)


def test_resident_fp32_matrix_sizes(cuda):
    from paper_1107_0538_amd import Solver

    for n in (40, 5000, 30000):
        a = banded(n, (1, 20), seed=n)
        b = np.random.default_rng(n).uniform(-1, 1, n)
        x, info = Solver(a, fp32_copy=True).solve_mixed_matrix(_t(b, cuda))
        xo, _ = oracle.pcg(a, b)
        assert info["status"] == 0 and oracle.relres(a, b, x.cpu().numpy()) <= tol_recomputed(n)
        assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-8 * np.linalg.norm(xo)


def test_resident_solves_from_several_threads(cuda):
    # Solvers on streams of their own, called at the same time: each gets the
    # bits it gets alone.
    import torch

    from paper_1107_0538_amd import Solver

    jobs = []
    for i, n in enumerate((16, 31, 24)):
        a, b = W.problem(n, i)
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            bt = _t(b, cuda)
            s = Solver(a, stream=st)
            alone, _ = s.solve(bt)
        st.synchronize()
        jobs.append((s, st, bt, alone.clone()))
    torch.cuda.synchronize()
    bad = []

    def work(s, st, bt, alone):
        with torch.cuda.stream(st):
            for _ in range(5):
                x, info = s.solve(bt)
                if info["status"] != 0 or not torch.equal(x, alone):
                    bad.append(info)

    threads = [threading.Thread(target=work, args=j) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


@pytest.mark.parametrize("sizes,long_row", [
    ((1, 64, 65, 700, 3000), False),           # small: all systems on the card at once
    ((100,) * 40 + (33000, 5, 20000), False),  # more than one XCD, many teams
    ((60000,) * 5 + (130000, 1000), False),    # systems that queue for the card
    ((500, 600), True),                        # a row that is too long: the general path
])
def test_resident_batches(cuda, sizes, long_row):
    from paper_1107_0538_amd import Batch

    mats = [banded(n, (1, 30), seed=i) for i, n in enumerate(sizes)]
    if long_row:
        mats[1] = banded(sizes[1], tuple(range(1, 16)), seed=9)
    rng = np.random.default_rng(len(sizes))
    bs = [rng.uniform(-1, 1, a.n) for a in mats]
    bt = Batch(mats)
    x, infos = bt.solve(_t(np.concatenate(bs), cuda))
    y, infos2 = bt.solve(_t(np.concatenate(bs), cuda))
    assert np.array_equal(x.cpu().numpy(), y.cpu().numpy())
    x = x.cpu().numpy()
    for s, a in enumerate(mats):
        check(a, bs[s], x[bt.offsets[s]:bt.offsets[s + 1]], infos[s], "standard")
    x, infos = bt.solve(_t(np.concatenate(bs), cuda), maxit=2)
    assert all(i["iters"] <= 2 for i in infos) and all(i["status"] == (0 if a.n <= 2 else 1) for i, a in zip(infos, mats))
