"""A sweep in one launch whose bounded wait runs out (forced by a limit of one
look) ends every entry point with its own error, not with NaN or an error that
blames the input, and leaves nothing behind: with the library's limit back, the
results are those of before bit for bit."""
import numpy as np
import pytest
import torch

from paper_2208_08594_amd import msp, synth

pytestmark = pytest.mark.gpu

STALL = -11
# (options, stages that sweep): block ILU(0) in the natural order; coarse
# Gauss-Seidel sweeps (one each way); both; an apply captured into a graph
CASES = {
    "bilu": (dict(max_coarse=10000, bilu_order=0), ("apply", "bilu_apply")),
    "bilu-fp32": (dict(max_coarse=10000, bilu_order=0, precond_fp32=True),
                  ("apply", "bilu_apply")),
    "gs": (dict(max_coarse=300), ("apply", "vcycle")),
    "both": (dict(max_coarse=300, bilu_order=0), ("apply", "vcycle", "bilu_apply")),
    "captured": (dict(max_coarse=300, bilu_order=0, n_stage=1, nu_pre=8, nu_post=8),
                 ("apply", "bilu_apply")),
}


def stalls(f):
    with pytest.raises(msp.MspError) as e:
        f()
    assert e.value.code == STALL


@pytest.mark.parametrize("name", sorted(CASES))
def test_wait_that_runs_out(name):
    opt, stages = CASES[name]
    s = synth.lognormal_grid(30, 26, 24, 3, 12, 1.5, 0.1, "lateral4")
    print("[case]", name, s.n, flush=True)
    g = msp.Solver(**opt)
    g.setup(s)
    rng = np.random.default_rng(4)
    v, f = rng.uniform(-1, 1, s.N), rng.uniform(-1, 1, s.n)
    x, info = g.solve(s.rhs)
    ref = {k: getattr(g, k)(f if k == "vcycle" else v) for k in stages}
    rhs = torch.as_tensor(s.rhs, device="cuda")
    for rep in range(2):
        g.set_limit(msp.LIMIT_SWEEP_POLLS, 1)
        for k in stages:
            stalls(lambda: getattr(g, k)(f if k == "vcycle" else v))
        stalls(lambda: g.solve(s.rhs))
        stalls(lambda: g.solve(s.rhs, noalloc=True))
        stalls(lambda: msp.solve_batch([g], [rhs], [torch.zeros_like(rhs)]))
        out = torch.zeros_like(rhs)
        stalls(lambda: g.repeat(msp.STAGE_PRECOND, 2, rhs, out))
        g.spmv(v)  # no sweep: no error left over
        g.set_limit(msp.LIMIT_SWEEP_POLLS, 0)
        for k in stages:
            assert torch.equal(getattr(g, k)(f if k == "vcycle" else v), ref[k])
        y, info2 = g.solve(s.rhs)
        assert info2["status"] == 0 and info2["iterations"] == info["iterations"]
        assert torch.equal(x, y)
    g.close()


def test_a_non_finite_right_hand_side_keeps_its_error():
    s = synth.lognormal_grid(20, 16, 12, 3, 12, 1.5, 0.1, "lateral4")
    g = msp.Solver(max_coarse=300, bilu_order=0)
    g.setup(s)
    rhs = s.rhs.copy()
    rhs[5] = np.nan
    with pytest.raises(msp.MspError) as e:
        g.solve(rhs)
    assert e.value.code == -4
    g.close()
