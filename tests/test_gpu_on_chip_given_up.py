"""On-chip solves in which a workgroup gives up waiting.

Every wait of the on-chip kernels is bounded.  Whatever the other workgroups
have seen and written by then, the host takes nothing of such a launch: x goes
back to what the caller passed and the general kernels solve the system, so
the result is bitwise that of a context made for them.  A workgroup that is
not there keeps the others waiting for as long as they may (a millisecond
here); one that gives up as the others finish, its last look having come before
words that they have seen, tells the host alone.
"""
import ctypes

import numpy as np
import pytest

import oracle
import workloads as W
from conftest import tol_recomputed
from test_gpu_resident import banded

pytestmark = pytest.mark.gpu


def _t(a, dev):
    import torch

    return torch.as_tensor(np.ascontiguousarray(a), device=dev)


@pytest.fixture
def on_chip(cuda):
    """on_chip(wait_limit, absent, given_up) sets the conditions for this thread's calls (-1, 0, 0: as ever)."""
    from paper_1107_0538_amd import capi

    f = capi.load().jpcg_test_on_chip
    f.argtypes, f.restype = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int], None
    yield f
    f(-1, 0, 0)


def solved_on_chip(s):
    from paper_1107_0538_amd import capi

    f = capi.load().jpcg_test_solved_on_chip
    f.argtypes, f.restype = [ctypes.c_void_p], ctypes.c_int
    return f(s.ctx)


def batch_solved_on_chip(bt):
    from paper_1107_0538_amd import capi

    f = capi.load().jpcg_test_batch_solved_on_chip
    f.argtypes, f.restype = [ctypes.c_void_p], ctypes.c_int
    return f(bt.h)


MS = 100000  # device ticks
HOW = {"one absent": (MS, 1, 0), "one gave up at the end": (-1, 0, 1), "nobody": (-1, 0, 0)}


@pytest.mark.parametrize("how", list(HOW))
@pytest.mark.parametrize("form", ["standard", "single", "fp32"])
@pytest.mark.parametrize("n,offsets", [(60, (1,)), (4000, (1, 30)), (30000, (1, 150))])  # one workgroup, group, eight
def test_given_up_solve_is_done_again(cuda, on_chip, n, offsets, form, how):
    from paper_1107_0538_amd import Solver

    a = banded(n, offsets, seed=n)
    rng = np.random.default_rng(n)
    b, x0 = _t(rng.uniform(-1, 1, n), cuda), _t(rng.uniform(-1, 1, n), cuda)
    kw = dict(form="single") if form == "single" else dict(fp32_copy=form == "fp32")

    def solve(s):
        return (s.solve_mixed_matrix if form == "fp32" else s.solve)(b, x0=x0)

    # A chunk length keeps the reference off the chip (16 and 8 are the
    # defaults), 32-bit columns off the slices, which small systems have not.
    ref, iref = solve(Solver(a, chunk=8 if form == "fp32" else 16, col_bits=32, **kw))
    s = Solver(a, **kw)
    alone, _ = solve(s)
    assert solved_on_chip(s) == 1
    on_chip(*HOW[how])
    x, info = solve(s)
    expected = how == "nobody" or (n == 60 and how == "one absent")  # alone, and there
    assert solved_on_chip(s) == int(expected)
    if expected:
        assert (x == alone).all()
    else:
        assert (x == ref).all() and (info["iters"], info["status"]) == (iref["iters"], iref["status"])
    on_chip(-1, 0, 0)
    x, _ = solve(Solver(a, **kw))
    assert (x == alone).all()


@pytest.mark.parametrize("how", list(HOW))
def test_given_up_batch_is_done_again(cuda, on_chip, how):
    from paper_1107_0538_amd import Batch

    mats = [banded(n, (1, 30), seed=i) for i, n in enumerate((700, 3000, 65, 20000))]
    rng = np.random.default_rng(4)
    total = sum(a.n for a in mats)
    b, x0 = _t(rng.uniform(-1, 1, total), cuda), _t(rng.uniform(-1, 1, total), cuda)
    ref, iref = Batch(mats, nnz_per_lane=16).solve(b, x0=x0)
    bt = Batch(mats)
    alone, _ = bt.solve(b, x0=x0)
    assert batch_solved_on_chip(bt) == 1
    on_chip(*HOW[how])
    x, info = bt.solve(b, x0=x0)
    assert batch_solved_on_chip(bt) == int(how != "one gave up at the end")
    if how != "one gave up at the end":  # a batch is launched whole
        assert (x == alone).all()
    else:
        assert (x == ref).all() and [i["iters"] for i in info] == [i["iters"] for i in iref]
    on_chip(-1, 0, 0)
    x, _ = Batch(mats).solve(b, x0=x0)
    assert (x == alone).all()


def test_batch_waits_for_earlier_systems(cuda, on_chip):
    # Systems that queue for the card, two of three solved in a tenth of the
    # iterations: a team's first round lasts until its last workgroup is through
    # with the system before, over 1 ms in ten of them, while no other round may
    # take longer than 0.2 ms.
    from paper_1107_0538_amd import Batch

    mats, bs = [], []
    for i in range(32):
        a, b = W.problem(40 - i % 8, i)
        mats.append(banded(a.n, (1, 30), seed=i) if i % 3 else a)
        bs.append(b)
    b = _t(np.concatenate(bs), cuda)
    bt = Batch(mats)
    alone, ialone = bt.solve(b)
    assert batch_solved_on_chip(bt) == 1
    on_chip(MS // 5, 0, 0)
    x, info = bt.solve(b)
    assert batch_solved_on_chip(bt) == 1
    assert (x == alone).all() and [i["iters"] for i in info] == [i["iters"] for i in ialone]


def test_batch_reports_where_it_ran(cuda):
    from paper_1107_0538_amd import Batch

    a, rhs = W.problem(8, 0)
    bt = Batch([a, a])
    bt.solve(_t(np.concatenate([rhs, rhs]), cuda))
    assert batch_solved_on_chip(bt) == 1
    bt = Batch([a, a], nnz_per_lane=8)
    bt.solve(_t(np.concatenate([rhs, rhs]), cuda))
    assert batch_solved_on_chip(bt) == 0


def test_no_memory_for_the_on_chip_solver(cuda):
    # The on-chip solver is one way of several: contexts and batches are made
    # without it where its arrays find no memory.
    from paper_1107_0538_amd import Batch, Solver, capi

    a, b = W.problem(12, 0)
    no_memory = capi.load().jpcg_test_no_memory
    no_memory(1)
    try:
        s = Solver(a)
        bt = Batch([a, a])
    finally:
        no_memory(0)
    for x, info in (s.solve(_t(b, cuda)), Solver(a).solve(_t(b, cuda))):
        assert info["status"] == 0 and oracle.relres(a, b, x.cpu().numpy()) <= tol_recomputed(a.n)
    assert solved_on_chip(s) == 0
    x, infos = bt.solve(_t(np.concatenate([b, b]), cuda))
    assert batch_solved_on_chip(bt) == 0 and all(i["status"] == 0 for i in infos)
    assert (x[:a.n] == x[a.n:]).all() and oracle.relres(a, b, x[:a.n].cpu().numpy()) <= tol_recomputed(a.n)


def test_many_small_systems_take_little_memory(cuda):
    # Systems of one workgroup exchange no sums: 500 of them, with all their
    # arrays, in less than 16 MB.
    import torch

    from paper_1107_0538_amd import Batch

    a = banded(40, (1,), seed=3)
    Batch([a] * 8)  # what the library and the runtime take once
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    bt = Batch([a] * 500)
    held = free - torch.cuda.mem_get_info()[0]
    assert held < 16 << 20, held
    b = _t(np.random.default_rng(5).uniform(-1, 1, 40), cuda).repeat(500)
    x, infos = bt.solve(b)
    assert batch_solved_on_chip(bt) == 1 and all(i["status"] == 0 for i in infos)
    assert (x.view(500, 40) == x[:40]).all()
    assert oracle.relres(a, b[:40].cpu().numpy(), x[:40].cpu().numpy()) <= tol_recomputed(40)


@pytest.mark.parametrize("batch", [False, True])
def test_given_up_launches_are_not_tried_at_once_again(cuda, on_chip, batch):
    # One solve without a try after the first launch that is given up, then two,
    # and none once a launch succeeds.
    from paper_1107_0538_amd import Batch, Solver

    a = banded(4000, (1, 30), seed=7)
    b = _t(np.random.default_rng(8).uniform(-1, 1, a.n), cuda)
    s = Batch([a]) if batch else Solver(a)
    there = batch_solved_on_chip if batch else solved_on_chip

    def solve():
        x, info = s.solve(b)
        assert (info[0] if batch else info)["status"] == 0
        assert oracle.relres(a, b.cpu().numpy(), x.cpu().numpy()) <= tol_recomputed(a.n)
        return there(s)

    assert [solve(), solve()] == [1, 1]
    leaves = (-1, 0, 1)
    on_chip(*leaves)
    assert solve() == 0
    on_chip(-1, 0, 0)
    assert [solve(), solve(), solve()] == [0, 1, 1]
    on_chip(*leaves)
    assert [solve(), solve(), solve()] == [0, 0, 0]  # the third is a try
    on_chip(-1, 0, 0)
    assert [solve(), solve(), solve()] == [0, 0, 1]


@pytest.mark.parametrize("edges", [(53, 20), (54, 20), (64, 20), (64, 54, 53, 64)])
def test_batch_halo_of_large_lattices(cuda, edges):
    # 512 rows of a 27-point lattice refer to 1332 others at 53^3, 1354 at 54^3
    # and 1408 at 64^3: three, then four for a thread.
    from paper_1107_0538_amd import Batch, Solver

    probs = [W.problem(n, i) for i, n in enumerate(edges)]
    bt = Batch([p[0] for p in probs])
    x, infos = bt.solve(_t(np.concatenate([p[1] for p in probs]), cuda))
    assert batch_solved_on_chip(bt) == 1
    for s, (a, b) in enumerate(probs):
        xs = x[bt.offsets[s]:bt.offsets[s + 1]]
        xo, io = Solver(a).solve(_t(b, cuda))
        assert infos[s]["status"] == io["status"] == 0 and abs(infos[s]["iters"] - io["iters"]) <= 2
        assert oracle.relres(a, b, xs.cpu().numpy()) <= tol_recomputed(a.n)
        assert float((xs - xo).norm() / xo.norm()) <= 1e-8
