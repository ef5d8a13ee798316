"""A nested-dissection factorisation that fails its check gives way to the
natural-order solver within the same setup, and the next setup on the pattern
starts with nested dissection again."""
import numpy as np
import pytest
import torch

import _checks as K
from oracle import oracle as O
from paper_2208_08594_amd import msp, synth

pytestmark = pytest.mark.gpu


# the whole matrix is the coarsest level; a hierarchy of several levels, on the
# device and on the host
@pytest.mark.parametrize("opt", [dict(max_coarse=10000), dict(max_coarse=1500),
                                 dict(max_coarse=1500, host_chain=True),
                                 dict(max_coarse=1500, precond_fp32=True),
                                 dict(max_coarse=1500, n_stage=1, bilu_order=0)])
def test_rejected_factorisation(opt):
    s = synth.lognormal_grid(23, 17, 12, 3, 6, 1.5, 0.1, "lateral4")
    print("[case]", opt, flush=True)
    fresh = msp.Solver(**opt)
    fresh.setup(s)
    f = np.random.default_rng(1).uniform(-1, 1, s.n)
    e, (x, info) = fresh.vcycle(f), fresh.solve(s.rhs)
    nL = fresh.info()["level_rows"][-1]
    bytes_nd = fresh._alloc.bytes_live

    o = O.OracleSolver(**{k: v for k, v in opt.items() if k != "host_chain"})
    o.setup(s)
    fp32 = opt.get("precond_fp32", False)
    t = 1e-5 if fp32 else K.coarse_tol_of(o.level(o.nlevels - 1))

    g = msp.Solver(**opt)
    for rep in range(2):
        g.set_limit(msp.LIMIT_ND_REJECTS, 1)
        assert g.setup(s)
        # the natural order holds two dense triangles
        g.solve(s.rhs)
        assert g._alloc.bytes_live > bytes_nd + 8 * nL * nL
        K.close(g.vcycle(f).cpu().numpy(), o.vcycle(f), t, "V-cycle, natural order")
        y, info2 = g.solve(s.rhs)
        assert info2["status"] == 0 and info2["iterations"] == info["iterations"]
        # the next setup: as a context that never fell back
        assert g.setup(s)
        assert torch.equal(g.vcycle(f), e)
        z, _ = g.solve(s.rhs)
        assert torch.equal(z, x) and g._alloc.bytes_live == bytes_nd
    g.close()
    fresh.close()
    o.close()
