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
