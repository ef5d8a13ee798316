"""The nested-dissection coarsest-level solver: its plan carried out on the
host (every stored index range checked) against a dense solve, which patterns
and matrices it declines, and on the GPU the direct solve against the oracle's
at the edges of its tiles, leaves and node sizes.

Tolerances: the plan's solve and the GPU's are held to the componentwise
backward error |A x - f| <= t (|A| |x| + |f|) with t = kappa(A) 1e-15 clipped
to [1e-12, 1e-10], the bar of every stage that includes the coarsest solve.
"""
import ctypes as C
import os
import subprocess
import tempfile

import numpy as np
import pytest
import scipy.sparse as sp

import _checks as K
from paper_2208_08594_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2208_08594_amd", "csrc")


@pytest.fixture(scope="module")
def shim():
    d = tempfile.mkdtemp()
    so = os.path.join(d, "libndshim.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-pthread", f"-I{CSRC}",
                           os.path.join(ROOT, "tests", "native", "nd_shim.cpp"),
                           os.path.join(CSRC, "msp_nd.cpp"), "-o", so])
    L = C.CDLL(so)
    i32 = np.ctypeslib.ndpointer(np.int32, flags="C")
    f64 = np.ctypeslib.ndpointer(np.float64, flags="C")
    L.shim_nd_solve.argtypes = [C.c_int, i32, i32, f64, f64, f64, C.POINTER(C.c_longlong)]
    return L


def dominant(A, seed, margin=0.05):
    """Random values on A's pattern (both signs, not symmetric) with every row
    dominant by `margin`."""
    rng = np.random.default_rng(seed)
    A = sp.csr_matrix(A, copy=True)
    A.setdiag(1.0)
    A.sort_indices()
    n = A.shape[0]
    rows = np.repeat(np.arange(n), np.diff(A.indptr))
    A.data = rng.uniform(-1.0, 1.0, A.nnz)
    d = rows == A.indices
    off = np.bincount(rows, weights=np.where(d, 0.0, np.abs(A.data)), minlength=n)
    A.data[d] = (off + 0.1) * (1.0 + margin) * rng.choice([-1.0, 1.0], n)[rows[d]]
    return A


def grid(nx, ny, nz):
    rp, ci, v = synth.poisson_csr((nx, ny, nz))
    return sp.csr_matrix((v, ci, rp), shape=(nx * ny * nz,) * 2)


def two_rings(A):
    """The pattern of A^2: the wider stencils of aggregated levels."""
    B = (abs(A) @ abs(A)).tocsr()
    B.data[:] = 1.0
    return B


def parts(*ms):
    return sp.block_diag(ms, format="csr")


PATTERNS = {
    "one": lambda: grid(1, 1, 1),
    "chain63": lambda: grid(63, 1, 1),
    "chain64": lambda: grid(64, 1, 1),
    "chain65": lambda: grid(65, 1, 1),
    "leaf128": lambda: grid(8, 4, 4),
    "leaf129": lambda: grid(43, 3, 1),
    "chain700": lambda: grid(700, 1, 1),
    "cube11": lambda: grid(11, 11, 11),
    "slab": lambda: grid(40, 17, 3),
    "wide14": lambda: two_rings(grid(14, 13, 6)),
    "islands": lambda: parts(grid(9, 9, 5), grid(1, 1, 1), grid(3, 1, 1), grid(150, 1, 1),
                             grid(1, 1, 1), grid(5, 5, 5)),
    "diagonal": lambda: sp.identity(200, format="csr"),
}


def permuted(A, seed):
    p = np.random.default_rng(seed).permutation(A.shape[0])
    A = A[p][:, p].tocsr()
    A.sort_indices()
    return A


def args(A):
    return (A.shape[0], np.ascontiguousarray(A.indptr, dtype=np.int32),
            np.ascontiguousarray(A.indices, dtype=np.int32), np.ascontiguousarray(A.data))


def tol_of(A):
    return max(1e-12, min(1e-10, np.linalg.cond(A.toarray()) * 1e-15))


@pytest.mark.parametrize("order", ["natural", "shuffled"])
@pytest.mark.parametrize("name", sorted(PATTERNS))
def test_plan_solves(shim, name, order):
    A = dominant(PATTERNS[name](), 3)
    if order == "shuffled":
        A = permuted(A, 4)
    f = np.random.default_rng(5).uniform(-1, 1, A.shape[0])
    x = np.zeros_like(f)
    ent = C.c_longlong()
    assert shim.shim_nd_solve(*args(A), f, x, C.byref(ent)) == 0
    K.dense_backward_error(A, x, f, tol_of(A), name)
    if name in ("cube11", "chain700", "slab"):
        assert ent.value < 0.5 * A.shape[0] ** 2


def test_plan_declines(shim):
    ent = C.c_longlong()
    A = dominant(grid(6, 5, 4), 1)
    f = np.ones(A.shape[0])
    x = np.zeros_like(f)
    # one row short of strict dominance
    B = A.copy()
    B[17, 17] = (abs(B[17]).sum() - abs(B[17, 17])) * (1.0 + 0.9e-5)
    assert shim.shim_nd_solve(*args(B), f, x, C.byref(ent)) == 2
    # not structurally symmetric, in a lower or in an upper entry
    for i, j in ((100, 3), (3, 100)):
        B = A.tolil()
        B[i, j] = 1e-3
        B[i, i] = B[i, i] * 2
        B = B.tocsr()
        B.sort_indices()
        assert shim.shim_nd_solve(*args(B), f, x, C.byref(ent)) == 1
    # a graph that does not separate: one dense block
    n = 1100
    B = dominant(sp.csr_matrix(np.ones((n, n))), 2)
    f = np.ones(n)
    assert shim.shim_nd_solve(*args(B), f, np.zeros(n), C.byref(ent)) == 1


# --------------------------------------------------------------------------
# GPU
# --------------------------------------------------------------------------
@pytest.mark.gpu
@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("name", sorted(PATTERNS))
def test_gpu_direct_solve(name, fp32):
    """The whole matrix is the coarsest level, so the V-cycle is the direct
    solve alone: against the oracle's LAPACK solve, and row by row."""
    from oracle import oracle as O
    from paper_2208_08594_amd import msp
    A = dominant(PATTERNS[name](), 7)
    # the decoupled level 0 of a scalar system is D^-1 A
    n, rp, ci, v = args(A)
    print("[case]", name, fp32, n, flush=True)
    g = msp.Solver(max_coarse=10000, precond_fp32=fp32)
    o = O.OracleSolver(max_coarse=10000)
    f = np.random.default_rng(8).uniform(-1, 1, n)
    for step in range(2):  # the second setup keeps the plan of the pattern
        vals = (v * (1.0 + 0.01 * step)).reshape(-1, 1, 1)
        g.setup(n=n, b=1, p=0, row_ptr=rp, col_ind=ci, vals=vals)
        o.setup(n=n, b=1, p=0, row_ptr=rp, col_ind=ci, vals=vals)
        assert o.nlevels == 1 and g.nlevels == 1
        x = g.vcycle(f).cpu().numpy()
        Lc = K.csr(o.level(0))
        t = tol_of(Lc)
        if fp32:  # f and x are rounded to FP32; the solve itself is FP64
            f32 = f.astype(np.float32).astype(np.float64)
            xo = o.vcycle(f32)
            K.assert_entrywise(x, xo, 2.0 ** -24 * 1.01, np.abs(xo) + 1e-30 + t * np.abs(xo).max() * 2.0 ** 24, name)
        else:
            K.dense_backward_error(Lc, x, f, t, name)
            K.close(x, o.vcycle(f), t, name)
        xs, info = g.solve(f, rtol=1e-8)
        assert info["rel_true_residual"] <= 1e-8
    g.close()
    o.close()


@pytest.mark.gpu
def test_gpu_both_solvers_agree_below_a_smoothed_level():
    """A two-level hierarchy whose coarsest level is served in nested
    dissection order: V-cycle and apply against the oracle, natural order of
    the finer level throughout."""
    from oracle import oracle as O
    from paper_2208_08594_amd import msp
    sys_ = synth.lognormal_grid(23, 17, 12, 3, 6, 1.5, 0.1, "lateral4")
    g = msp.Solver(max_coarse=1500)
    o = O.OracleSolver(max_coarse=1500)
    g.setup(sys_)
    o.setup(sys_)
    assert g.nlevels == o.nlevels == 2
    t = K.coarse_tol_of(o.level(1))
    f = np.random.default_rng(1).uniform(-1, 1, sys_.n)
    K.close(g.vcycle(f).cpu().numpy(), o.vcycle(f), t, "V-cycle")
    v = np.random.default_rng(2).uniform(-1, 1, sys_.N)
    K.close(g.apply(v).cpu().numpy(), o.apply(v), t, "apply")
    g.close()
    o.close()
