"""Block products and triangular solves on both sides of the slice counts at
which they change between a wave per component and a wave per slice: A x to
1e-13 of (|A| |x|) row by row against scipy, the block ILU(0) solve to 1e-12
(FP32 apply 1e-5) of its largest entry against the oracle, the bars of
test_component_split.py."""
import numpy as np
import pytest
import scipy.sparse as sp

import _checks as K
from oracle import oracle as O
from paper_2208_08594_amd import msp, synth

pytestmark = pytest.mark.gpu


# slices of 64 rows: 1536, 1537, 1600, 1350, 1400, 2048, 2049, 2200
@pytest.mark.parametrize("dims,b", [((64, 48, 32), 3), ((53, 58, 32), 3), ((64, 50, 32), 4),
                                    ((64, 54, 25), 6), ((64, 50, 28), 6), ((64, 64, 32), 4),
                                    ((683, 64, 3), 4), ((64, 55, 40), 6)])
def test_product(dims, b):
    s = synth.lognormal_grid(*dims, b, 3, 1.0, 1.0, "corners2")
    print("[case]", dims, b, (s.n + 63) // 64, flush=True)
    g = msp.Solver(max_coarse=10000)
    g.setup(s)
    x = np.random.default_rng(b).uniform(-1, 1, s.N)
    A = sp.bsr_matrix((s.vals, s.col_ind, s.row_ptr), shape=(s.N, s.N))
    K.assert_entrywise(g.spmv(x).cpu().numpy(), A @ x, 1e-13, abs(A) @ np.abs(x), "A x")
    g.close()


# levels of 1550 and 1600 slices (FP64), of 1300 and 1350 (FP32)
@pytest.mark.parametrize("dims,b,fp32", [((64, 62, 50), 4, False), ((64, 64, 50), 4, False),
                                         ((64, 52, 50), 4, True), ((64, 54, 50), 4, True)])
def test_solve(dims, b, fp32):
    s = synth.lognormal_grid(*dims, b, 3, 1.0, 1.0, "corners2")
    print("[case]", dims, b, fp32, (s.n // 2 + 63) // 64, flush=True)
    g = msp.Solver(max_coarse=10000, precond_fp32=fp32)
    o = O.OracleSolver(max_coarse=10000, precond_fp32=fp32)
    g.setup(s)
    o.setup(s)
    r = np.random.default_rng(b).uniform(-1, 1, s.N)
    zo = o.apply(r) if fp32 else o.bilu_apply(r)
    z = (g.apply(r) if fp32 else g.bilu_apply(r)).cpu().numpy()
    K.assert_entrywise(z, zo, 1e-5 if fp32 else 1e-12, np.abs(zo).max(), "solve")
    g.close()
    o.close()
