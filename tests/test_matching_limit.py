"""The matching's bounded runs: whatever the limit of a row's looks at undecided
rows, every run decides some row and the aggregates are those of the ascending
pass, also where a row walks along many more taken candidates or in-rows than
the limit (those looks end with the lists and are not counted)."""
import ctypes as C
import os
import subprocess
import tempfile

import numpy as np
import pytest
import scipy.sparse as sp

from oracle import oracle as O
from paper_2208_08594_amd import msp
from test_matching import chain, hubs, laplacian, random_ties

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2208_08594_amd", "csrc")


def taken(m):
    """Rows 0..m-1 take m+1..2m; row m between them has all of those, taken by
    then, as its candidates."""
    i = np.arange(m)
    return laplacian(sp.csr_matrix(sp.coo_matrix(
        (np.r_[np.ones(m), np.full(m, 0.5)], (np.r_[i, np.full(m, m)], np.r_[i, i] + m + 1)),
        shape=(2 * m + 1,) * 2)))


def crowded(m, k):
    """As taken(m), and every candidate has k more in-rows below row m, which
    pair among themselves (the taker is the last of the in-rows looked at)."""
    n = m + 2 * k + 1 + m
    w = m + 2 * k
    W = sp.lil_matrix((n, n))
    for q in range(k):
        W[m + 2 * q, m + 2 * q + 1] = 1.0
        for i in range(m):
            W[m + 2 * q, w + 1 + i] = 0.5
    for i in range(m):
        W[i, w + 1 + i] = 1.0
        W[w, w + 1 + i] = 0.5
    return laplacian(W)


CASES = {
    "chain1025": lambda: chain(1025),
    "ties2049": lambda: random_ties(2049, 2, 1),
    "ties900-dense": lambda: random_ties(900, 9, 2),
    "hubs2500": lambda: hubs(2500, 3),
    "taken3": lambda: taken(3),
    "taken200": lambda: taken(200),
    "taken1500": lambda: taken(1500),
    "crowded12x40": lambda: crowded(12, 40),
}
LIMITS = [1, 2, 5, 64]


def csr(A):
    return (A.shape[0], np.ascontiguousarray(A.indptr, dtype=np.int32),
            np.ascontiguousarray(A.indices, dtype=np.int32), np.ascontiguousarray(A.data))


@pytest.fixture(scope="module")
def shim():
    d = tempfile.mkdtemp()
    so = os.path.join(d, "libmatchshim.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-pthread",
                           "-ffp-contract=off", "-Wno-unknown-pragmas", f"-I{CSRC}",
                           os.path.join(ROOT, "tests", "native", "match_shim.cpp"),
                           os.path.join(CSRC, "msp_host.cpp"), "-o", so])
    L = C.CDLL(so)
    i32 = np.ctypeslib.ndpointer(np.int32, flags="C")
    f64 = np.ctypeslib.ndpointer(np.float64, flags="C")
    L.shim_match.argtypes = [C.c_int, i32, i32, f64, C.c_int, C.c_int, i32]
    L.shim_pairwise.argtypes = [C.c_int, i32, i32, f64, i32]
    return L


@pytest.mark.parametrize("up", [0, 1])
@pytest.mark.parametrize("name", sorted(CASES))
def test_every_run_decides(shim, name, up):
    A = csr(CASES[name]())
    ref = np.zeros(A[0], dtype=np.int32)
    shim.shim_pairwise(*A, ref)
    for looks in LIMITS + [32768]:
        agg = np.zeros_like(ref)
        runs = shim.shim_match(*A, looks, up, agg)
        assert runs > 0, (name, looks)
        assert np.array_equal(agg, ref), (name, looks)
    if name.startswith(("taken", "crowded")):
        assert runs == 1  # nothing there waits for long


@pytest.mark.gpu
@pytest.mark.parametrize("looks", LIMITS)
@pytest.mark.parametrize("name", sorted(CASES))
def test_gpu_aggregates(name, looks):
    n, rp, ci, v = csr(CASES[name]())
    print("[case]", name, looks, n, flush=True)
    g = msp.Solver(max_coarse=40 if n > 60 else 2)
    o = O.OracleSolver(max_coarse=40 if n > 60 else 2)
    g.set_limit(msp.LIMIT_MATCH_LOOKS, looks)
    for s in (g, o):
        s.setup(n=n, b=1, p=0, row_ptr=rp, col_ind=ci, vals=v.reshape(-1, 1, 1).copy())
    assert g.nlevels == o.nlevels >= 2
    for l in range(o.nlevels):
        a, b = g.level(l), o.level(l)
        assert np.array_equal(a["col_ind"], b["col_ind"])
        assert np.array_equal(a["val"], b["val"])
        if l + 1 < o.nlevels:
            assert np.array_equal(a["agg"], b["agg"])
    g.close()
    o.close()
