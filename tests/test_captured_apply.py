"""The preconditioner apply captured into a graph (more launches than are
launched one by one) against the same kernels launched eagerly, bit for bit: on
every replay, after a setup that keeps the preconditioner, after one with other
values that regenerates it, after one with another pattern, and in the form of
the concentration stage, whose vectors are copied in and out."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2208_08594_amd import msp, synth

pytestmark = pytest.mark.gpu

# eight sweeps each way: some 200 launches with the levels of max_coarse = 300
MANY = dict(max_coarse=300, nu_pre=8, nu_post=8)
CASES = {
    "default": {},
    "fp32": dict(precond_fp32=True),
    "jacobi": dict(smoother=1, nu_pre=8, nu_post=8, bilu_order=0, jacobi_weight=0.7),
    "natural": dict(bilu_order=0),
    "block-jacobi": dict(full_smoother=1),
    "nstage": dict(n_stage=1),
    "nstage-natural": dict(n_stage=1, bilu_order=0),
    "nstage-natural-fp32": dict(n_stage=1, bilu_order=0, precond_fp32=True),
}


def perturbed(s, seed):
    rng = np.random.default_rng(seed)
    return dataclasses.replace(s, vals=s.vals * (1.0 + 0.05 * rng.uniform(-1, 1, s.vals.shape)))


def replays(ge, gg, s, rng):
    for rep in range(4):
        v = rng.uniform(-1, 1, s.N)
        ze, zg = ge.apply(v), gg.apply(v)
        gg.spmv(v)  # eager work between replays
        torch.cuda.synchronize()
        assert torch.equal(ze, zg), rep
    xe, ie = ge.solve(s.rhs)
    xg, ig = gg.solve(s.rhs)
    assert ie["iterations"] == ig["iterations"] and torch.equal(xe, xg)
    xn, _ = gg.solve(s.rhs, noalloc=True)
    assert torch.equal(xe, xn)


@pytest.mark.parametrize("name", sorted(CASES))
def test_replays_match_eager(name):
    opt = {**MANY, **CASES[name]}
    s = synth.lognormal_grid(28, 24, 20, 4, 12, 1.5, 0.1, "lateral4")
    other = synth.lognormal_grid(22, 26, 18, 4, 5, 1.5, 0.1, "lateral4")
    print("[case]", name, flush=True)
    # mu = 0: every setup regenerates; mu = 1000: every later one keeps B
    for mu in (0, 1000):
        ge = msp.Solver(mu=mu, use_graphs=False, **opt)
        gg = msp.Solver(mu=mu, use_graphs=True, **opt)
        rng = np.random.default_rng(13)
        seen = []
        for step, sys_ in enumerate((s, s, perturbed(s, 1), other, s)):
            kept = [g.setup(sys_) for g in (ge, gg)]
            assert kept[0] == kept[1] == (mu == 0 or step in (0, 3, 4))
            if kept[0]:
                assert gg.apply_nodes() == 0  # the graph went with the preconditioner
            replays(ge, gg, sys_, rng)
            assert ge.apply_nodes() == 0
            seen.append(gg.apply_nodes())
        assert min(seen) > 60  # (a Jacobi sweep is one or two kernels on any level)
        ge.close()
        gg.close()


# Small systems: a graph from some 40 launches on (the host takes longer to launch
# them than the device to run them); large ones: from some 160 on.
@pytest.mark.parametrize("dims,opt,graph", [
    ((10, 10, 10), dict(), False),
    ((10, 10, 10), dict(max_coarse=64, nu_pre=2), True),
    ((10, 10, 10), dict(max_coarse=12, smoother=1), True),
    ((24, 24, 24), dict(max_coarse=1500), False),
    ((24, 24, 24), dict(max_coarse=1500, nu_pre=4, nu_post=4), True),
    ((48, 48, 32), dict(max_coarse=3000, nu_pre=2, nu_post=1), False),
    ((48, 48, 32), dict(max_coarse=300, nu_pre=8, nu_post=8), True)])
def test_which_applies_are_captured(dims, opt, graph):
    s = synth.lognormal_grid(*dims, 4, 12, 1.5, 0.1, "lateral4")
    g = msp.Solver(**opt)
    e = msp.Solver(use_graphs=False, **opt)
    g.setup(s)
    e.setup(s)
    x, _ = g.solve(s.rhs)
    assert torch.equal(x, e.solve(s.rhs)[0])
    assert (g.apply_nodes() > 0) == graph
    if graph:
        assert g.apply_nodes() > (40 if s.N <= 262144 else 160)
    g.close()
    e.close()
