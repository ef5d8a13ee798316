"""Block products and triangular solves on both sides of the row count where a
slice changes from a wave per component to one wave: A x to 1e-13 of (|A| |x|)
row by row against scipy, the block ILU(0) solve to 1e-12 of its largest entry
against the oracle, as in test_gpu_parity.py."""
import numpy as np
import pytest
import scipy.sparse as sp

import _checks as K
from oracle import oracle as O
from paper_2208_08594_amd import msp, synth

pytestmark = pytest.mark.gpu


# the last two: 2500 and 2501 slices of 64 rows
@pytest.mark.parametrize("dims", [(1, 1, 2), (5, 4, 3), (13, 5, 1), (16, 8, 8), (50, 64, 50),
                                  (53, 61, 50)])
@pytest.mark.parametrize("b", [1, 2, 3, 4, 5, 6, 7, 8])
def test_product(dims, b):
    if b > 4 and np.prod(dims) > 10000 and b != 7:
        pytest.skip("large matrices with b = 1 to 4 and 7")
    s = synth.lognormal_grid(*dims, b, 3, 1.0, 1.0, "corners2")
    print("[case]", dims, b, flush=True)
    g = msp.Solver(max_coarse=10000)
    g.setup(s)
    x = np.random.default_rng(b).uniform(-1, 1, s.N)
    A = sp.bsr_matrix((s.vals, s.col_ind, s.row_ptr), shape=(s.N, s.N))
    scale = abs(A) @ np.abs(x)
    K.assert_entrywise(g.spmv(x).cpu().numpy(), A @ x, 1e-13, scale, "A x")
    g.close()


# levels of 2500 and of 2501 and more slices in the two-color order; chains of
# two rows; a remainder of one row
@pytest.mark.parametrize("dims,b", [((100, 64, 50), 1), ((101, 64, 50), 2), ((1, 1, 2), 4),
                                    ((13, 5, 1), 7), ((9, 8, 9), 8), ((16, 16, 9), 6)])
@pytest.mark.parametrize("fp32", [False, True])
def test_solve(dims, b, fp32):
    s = synth.lognormal_grid(*dims, b, 3, 1.0, 1.0, "corners2")
    print("[case]", dims, b, fp32, flush=True)
    g = msp.Solver(max_coarse=10000, precond_fp32=fp32)
    g.setup(s)
    o = O.OracleSolver(max_coarse=10000, precond_fp32=fp32)
    o.setup(s)
    r = np.random.default_rng(b).uniform(-1, 1, s.N)
    if fp32:
        zo = o.apply(r)
        K.assert_entrywise(g.apply(r).cpu().numpy(), zo, 1e-5, np.abs(zo).max(), "apply")
    else:
        zo = o.bilu_apply(r)
        K.assert_entrywise(g.bilu_apply(r).cpu().numpy(), zo, 1e-12, np.abs(zo).max(), "solve")
    g.close()
    o.close()
