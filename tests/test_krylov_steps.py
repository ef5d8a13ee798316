"""The Krylov part of the solve at the sizes where its launches change: the
reduction in a pass's last work-group (up to 786,432 unknowns) and in a launch
of its own beyond, restart lengths beyond the fused passes, steps queued ahead
of the host, and a captured preconditioner apply.  Against the oracle's iteration count and the true residual; repeated
solves bit for bit."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2208_08594_amd import msp, synth

pytestmark = pytest.mark.gpu


def true_residual(sys_, x):
    import _checks as K
    A = K.bsr(sys_)
    return np.linalg.norm(sys_.rhs - A @ x) / np.linalg.norm(sys_.rhs)


# unknowns: 1, 257, 1,024 and 1,025, near 256 work-groups of 1,024, and below, at
# and above the largest vector whose passes add up their own partials
SMALL = [((1, 1, 1), 1), ((257, 1, 1), 1), ((16, 8, 8), 1), ((41, 25, 1), 1)]
LARGE = [((64, 64, 32), 2), ((61, 61, 35), 2), ((64, 64, 64), 1), ((65, 64, 64), 1),
         ((64, 64, 64), 3), ((64, 48, 51), 5), ((61, 73, 59), 3)]


@pytest.mark.parametrize("dims,b,restart", [(d, b, m) for d, b in SMALL for m in (1, 5, 30, 40)] +
                         [(d, b, 30) for d, b in LARGE])
def test_solve_sizes(dims, b, restart):
    s = synth.lognormal_grid(*dims, b, 3, 1.0, 1.0, "none")
    print("[case]", dims, b, restart, flush=True)
    g = msp.Solver(restart=restart, max_iter=300)
    g.setup(s)
    x, info = g.solve(s.rhs, rtol=1e-9)
    assert info["status"] == 0 and info["rel_true_residual"] <= 1e-9
    xn = x.cpu().numpy()
    # recomputed with other rounding: within the accumulated rounding of one product
    assert true_residual(s, xn) <= 1e-9 * 1.01 + 1e-13
    x2, info2 = g.solve(s.rhs, rtol=1e-9)
    assert info2["iterations"] == info["iterations"] and torch.equal(x, x2)
    if np.prod(dims) <= 5000:
        o = O.OracleSolver(restart=restart, max_iter=300)
        o.setup(s)
        xo, it, rr, st = o.solve(s.rhs, 1e-9)
        assert abs(it - info["iterations"]) <= 1
        o.close()
    g.close()


@pytest.mark.parametrize("max_iter", [1, 2, 3, 7])
def test_steps_queued_ahead_stop_at_max_iter(max_iter):
    s = synth.config(0)
    g = msp.Solver(max_iter=max_iter, restart=5)
    g.setup(s)
    x, info = g.solve(s.rhs, rtol=1e-14)
    assert info["status"] == 1 and info["iterations"] == max_iter
    x2, _ = g.solve(s.rhs, rtol=1e-14)
    assert torch.equal(x, x2)
    g.close()


def test_initial_guess_and_exact_start():
    """A start at the solution needs no step; a start from another vector ends
    at the same solution."""
    s = synth.config(0)
    g = msp.Solver()
    g.setup(s)
    x, _ = g.solve(s.rhs, rtol=1e-12)
    y, info = g.solve(s.rhs, x.clone(), rtol=1e-10)
    assert info["iterations"] == 0 and torch.equal(x, y)
    z, info = g.solve(s.rhs, torch.ones_like(x), rtol=1e-12)
    assert info["iterations"] > 0
    assert float((z - x).norm() / x.norm()) <= 1e-9
    g.close()


@pytest.mark.parametrize("dims,b,opt", [
    ((5, 4, 3), 1, {}), ((10, 10, 10), 4, {}), ((24, 20, 11), 7, {"precond_fp32": True}),
    ((17, 13, 9), 3, {"bilu_order": 0}), ((17, 13, 9), 3, {"n_stage": 1}),
    ((61, 73, 59), 3, {})])
def test_scaled_basis_vector(dims, b, opt):
    """A new basis vector scaled inside the apply, and (as with events recorded
    around the parts) by a launch ahead of it: the same solve bit for bit."""
    s = synth.lognormal_grid(*dims, b, 3, 1.0, 1.0, "none")
    g = msp.Solver(**opt)
    g.setup(s)
    x, info = g.solve(s.rhs, rtol=1e-9)
    g.set_timing(True)
    y, info2 = g.solve(s.rhs, rtol=1e-9)
    assert info["iterations"] == info2["iterations"] and torch.equal(x, y)
    g.close()


@pytest.mark.parametrize("fp32", [False, True])
def test_captured_apply(fp32):
    """An apply of many launches is replayed from a graph: every replay equals
    the eager launches, with eager work between the replays."""
    s = synth.lognormal_grid(40, 33, 22, 3, 12, 1.5, 0.1, "lateral4")
    a = msp.Solver(max_coarse=300, nu_pre=8, nu_post=8, precond_fp32=fp32,
                   use_graphs=False)
    b = msp.Solver(max_coarse=300, nu_pre=8, nu_post=8, precond_fp32=fp32,
                   use_graphs=True)
    a.setup(s)
    b.setup(s)
    rng = np.random.default_rng(1)
    for rep in range(4):
        v = rng.uniform(-1, 1, s.N)
        za, zb = a.apply(v), b.apply(v)
        b.spmv(v)
        torch.cuda.synchronize()
        assert torch.equal(za, zb), rep
    xa, ia = a.solve(s.rhs)
    xb, ib = b.solve(s.rhs)
    assert ia["iterations"] == ib["iterations"] and torch.equal(xa, xb)
    a.close()
    b.close()
