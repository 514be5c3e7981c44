"""Block CG where its fused passes end: row counts at the edges of 16-row tiles and of the
workgroups' shares, one to 64 columns, a context used again with another width.

Each column's true residual meets the tolerance (the status says so on the recomputed residual) and
agrees with the single-system solve within 1e-8.
"""
import numpy as np
import pytest

import oracle
from conftest import tol_recomputed
from test_gpu_resident import banded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 127, 128, 129, 1023, 1025, 4099])
def test_block_rows(cuda, n):
    import torch

    from paper_1107_0538_amd import Solver

    a = banded(n, (1, 7) if n > 7 else (), seed=n)
    solver = Solver(a)
    for s in (1, 5, 64, 3):
        B = np.random.default_rng(n + s).uniform(-1, 1, (n, s))
        X, infos = solver.solve_block(torch.as_tensor(B, device=cuda))
        X = X.cpu().numpy()
        for j in range(0, s, 7):
            x, info = solver.solve(torch.as_tensor(np.ascontiguousarray(B[:, j]), device=cuda))
            assert infos[j]["status"] == info["status"] == 0
            assert oracle.relres(a, B[:, j], X[:, j]) <= tol_recomputed(n)
            assert np.linalg.norm(X[:, j] - x.cpu().numpy()) <= 1e-8 * np.linalg.norm(X[:, j])
