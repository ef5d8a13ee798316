"""Arnoldi steps are queued ahead of the host only where they are needed: a
large system that converges in a few steps queues just those, and a slow one at
most one more."""
import dataclasses

import numpy as np
import pytest

from paper_2208_08594_amd import msp, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grid():
    return synth.lognormal_grid(40, 40, 24, 4, 12, 1.5, 0.1, "lateral4")


def heavier(s, add):
    vals = s.vals.copy()
    vals[s.diag_pos] += add * np.eye(s.b)
    return dataclasses.replace(s, vals=vals)


@pytest.mark.parametrize("add,most", [(1e6, 1), (1e4, 1), (1e2, 2)])
def test_no_step_in_vain(grid, add, most):
    s = heavier(grid, add)
    g = msp.Solver()
    g.setup(s)
    for rep in range(2):
        x, info = g.solve(s.rhs)
        assert info["status"] == 0 and info["iterations"] <= most
        assert g.steps_queued() == info["iterations"]
    g.close()


@pytest.mark.parametrize("opt", [{}, dict(restart=4), dict(max_iter=3)])
@pytest.mark.parametrize("small", [False, True])
def test_at_most_one(grid, small, opt):
    s = synth.config(0) if small else grid
    g = msp.Solver(**opt)
    g.setup(s)
    x, info = g.solve(s.rhs, rtol=1e-8)
    # one at the end of each cycle at most, none beyond max_iter
    assert info["iterations"] <= g.steps_queued() <= info["iterations"] + info["restarts"]
    if "max_iter" in opt:
        assert g.steps_queued() == info["iterations"] == 3
    g.close()
