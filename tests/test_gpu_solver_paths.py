"""The solver's rarer paths through each of its kernels: residuals that are
replaced, and iteration limits at either parity, on chip, over slices and by
tiles.  The criteria are those of the single-system tests, against the oracle of
the same form; cg_get_config says that the kernels meant were the ones that ran.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from conftest import mean_removed_relerr, tol_recomputed
from test_gpu_kernel_paths import FORMS, ON_CHIP, SLICES, TILES, _t, kernels

pytestmark = pytest.mark.gpu

# Options that lead there: a chunk length keeps a system off the chip, 32-bit columns off the slices.
PATHS = {"on chip": (dict(), ON_CHIP), "slices": (dict(chunk=16), SLICES), "slices, odd chunks": (dict(chunk=7), SLICES),
         "tiles": (dict(chunk=16, col_bits=32), TILES), "tiles, odd chunks": (dict(chunk=7, col_bits=32), TILES)}


@pytest.mark.parametrize("path", list(PATHS))
@pytest.mark.parametrize("form", FORMS)
def test_replacement_below_attainable_accuracy(cuda, form, path):
    from paper_1107_0538_amd import Solver

    a, b = W.problem(16, 0)
    maxit = 400
    xo, io = oracle.pcg(a, b, tol=1e-16, maxit=maxit, form=form)
    opts, kind = PATHS[path]
    s = Solver(a, form=form, **opts)
    x, info = s.solve(_t(b, cuda), tol=1e-16, maxit=maxit)
    assert kernels(s)[0] == kind
    # The single-reduction form may also end in breakdown there, as the oracle does.
    assert io["status"] == info["status"] and (info["status"] == 1 or form == "single")
    if info["status"] == 1:
        assert info["iters"] == maxit
    assert io["replacements"] >= 1 and info["replacements"] >= 1
    assert info["relres_true"] <= 1e-10 and io["relres_true"] <= 1e-10
    assert np.linalg.norm(x.cpu().numpy() - xo) / np.linalg.norm(xo) <= 1e-6


@pytest.mark.parametrize("path", list(PATHS))
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("fam_n,first", [(14, 0), (16, 20)])
def test_converging_with_replacement(cuda, form, path, fam_n, first):
    from paper_1107_0538_amd import Solver

    a, _ = W.problem(fam_n, 0)
    fam = W.amplitude_family(n=fam_n, count=first + 10)
    opts, kind = PATHS[path]
    s = Solver(a, form=form, **opts)
    reps = 0
    for b in fam.rhs(np.arange(first, first + 8)):
        xo, io = oracle.pcg(a, b, form=form)
        x, info = s.solve(_t(b, cuda))
        assert kernels(s)[0] == kind
        reps += io["replacements"]
        assert info["status"] == io["status"] == 0, (info, io)
        assert abs(info["iters"] - io["iters"]) <= 2, (info, io)
        assert abs(info["replacements"] - io["replacements"]) <= 1, (info, io)
        assert np.linalg.norm(x.cpu().numpy() - xo) / np.linalg.norm(xo) <= 1e-8
        assert mean_removed_relerr(x.cpu().numpy(), xo) <= 1e-8
        assert oracle.relres(a, b, x.cpu().numpy()) <= tol_recomputed(a.n)
    assert reps >= 4


@pytest.mark.parametrize("path", list(PATHS))
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("maxit", [1, 2, 3, 16, 17, 33])
def test_iteration_limit(cuda, form, path, maxit):
    from paper_1107_0538_amd import Solver

    a, b = W.problem(16, 0)
    opts, kind = PATHS[path]
    s = Solver(a, form=form, **opts)
    x, info = s.solve(_t(b, cuda), maxit=maxit)
    assert kernels(s)[0] == kind
    xo, io = oracle.pcg(a, b, maxit=maxit, form=form)
    assert info["status"] == io["status"] == 1 and info["iters"] == io["iters"] == maxit
    assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-9 * np.linalg.norm(xo)
    assert abs(info["relres_true"] - io["relres_true"]) <= 1e-8 * io["relres_true"]
