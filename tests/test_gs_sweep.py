"""Coarse levels whose Gauss-Seidel sweeps run in one launch each, and the
restricted residual ahead of them: the V-cycle against the oracle's to
kappa(A_L) 1e-15 of its largest entry (the coarsest solve's bound, as in
test_gpu_parity.py), the FP32 apply to 1e-5."""
import numpy as np
import pytest
import torch

import _checks as K
from oracle import oracle as O
from paper_2208_08594_amd import msp, synth

pytestmark = pytest.mark.gpu

CASES = [
    # make, max_coarse, options of the solver
    (lambda: synth.lognormal_grid(40, 33, 22, 1, 12, 1.5, 0.1, "lateral4"), 60, {}),
    (lambda: synth.lognormal_grid(17, 13, 9, 3, 5, 1.0, 1.0, "corners2"), 20, {}),
    (lambda: synth.lognormal_grid(24, 24, 24, 2, 7, 1.5, 0.1, "lateral4"), 700, {}),
    # stalled coarsening: aggregates of many rows, long coarse rows
    (lambda: synth.layered_grid(20, 40, 15, 2, 1), 100, {}),
    # sweeps that the one-launch form does not cover
    (lambda: synth.layered_grid(20, 40, 15, 2, 1), 100, {"nu_post": 2}),
    (lambda: synth.lognormal_grid(17, 13, 9, 3, 5, 1.0, 1.0, "corners2"), 20, {"nu_pre": 2}),
    (lambda: synth.lognormal_grid(17, 13, 9, 3, 5, 1.0, 1.0, "corners2"), 20, {"nu_post": 0}),
]


@pytest.mark.parametrize("k", range(len(CASES)))
@pytest.mark.parametrize("fp32", [False, True])
def test_cycle(k, fp32):
    make, mc, opt = CASES[k]
    s = make()
    print("[case]", s.n, s.b, mc, opt, "fp32", fp32, flush=True)
    g = msp.Solver(max_coarse=mc, precond_fp32=fp32, **opt)
    g.setup(s)
    o = O.OracleSolver(max_coarse=mc, precond_fp32=fp32, **opt)
    o.setup(s)
    info = g.info()
    assert o.nlevels == g.nlevels >= 3 and max(info["n_colors"]) > 4
    f = np.random.default_rng(4).uniform(-1, 1, s.n)
    v = np.random.default_rng(5).uniform(-1, 1, s.N)
    if fp32:
        run, x = g.apply, v
        z, zo, tol = g.apply(v), o.apply(v), 1e-5
    else:
        run, x = g.vcycle, f
        z, zo, tol = g.vcycle(f), o.vcycle(f), K.coarse_tol_of(o.level(o.nlevels - 1))
    K.close(z.cpu().numpy(), zo, tol, "cycle")
    for rep in range(3):
        assert torch.equal(run(x), z)
    # a NaN or an infinity spreads, ends, and leaves nothing behind
    for bad in (np.nan, np.inf):
        y = x.copy()
        y[len(y) // 2] = bad
        assert not torch.isfinite(run(y)).all()
        assert torch.equal(run(x), z)
    g.close()
    o.close()
