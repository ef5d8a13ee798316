"""The pairwise matching of the device aggregation chain at the edges of its
work-groups (1,024 rows) and lists (records of four entries): aggregates and
coarse matrices bit for bit as the oracle's, on graphs with long dependency
chains, tied strengths and long candidate and in-row lists."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import oracle as O
from paper_2208_08594_amd import msp

pytestmark = pytest.mark.gpu


def laplacian(W):
    """Symmetric weights -> diagonally dominant scalar matrix with full diagonal."""
    W = sp.csr_matrix(W)
    W = W.maximum(W.T)
    W.setdiag(0.0)
    W.eliminate_zeros()
    A = sp.csr_matrix(sp.diags(np.asarray(W.sum(1)).ravel() + 0.5) - W)
    A.sort_indices()
    return A


def chain(n):
    return laplacian(sp.diags([np.ones(n - 1)], [1]))


def random_ties(n, deg, seed):
    """Random graph whose weights take four values (ties everywhere)."""
    rng = np.random.default_rng(seed)
    i = np.repeat(np.arange(n), deg)
    j = rng.integers(0, n, n * deg)
    w = rng.choice([0.25, 0.5, 0.75, 1.0], n * deg)
    return laplacian(sp.csr_matrix(sp.coo_matrix((w, (i, j)), shape=(n, n)).tocsr().minimum(1.0)))


def hubs(n, seed):
    """A chain with a few rows joined to hundreds of others, low and high."""
    rng = np.random.default_rng(seed)
    W = sp.lil_matrix(sp.diags([np.ones(n - 1)], [1]))
    for h in (0, 3, n // 2, n - 2):
        for j in rng.choice(n, 300, replace=False):
            if j != h:
                W[min(h, j), max(h, j)] = rng.choice([0.5, 1.0])
    return laplacian(W)


CASES = {
    "chain1023": lambda: chain(1023),
    "chain1024": lambda: chain(1024),
    "chain1025": lambda: chain(1025),
    "chain5000": lambda: chain(5000),
    "ties2049": lambda: random_ties(2049, 2, 1),
    "ties3000-dense": lambda: random_ties(3000, 9, 2),
    "hubs2500": lambda: hubs(2500, 3),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_matching_bit_exact(name):
    A = CASES[name]()
    n = A.shape[0]
    rp, ci = A.indptr.astype(np.int32), A.indices.astype(np.int32)
    vals = A.data.reshape(-1, 1, 1).copy()
    print("[case]", name, n, flush=True)
    g = msp.Solver(max_coarse=40)
    o = O.OracleSolver(max_coarse=40)
    g.setup(n=n, b=1, p=0, row_ptr=rp, col_ind=ci, vals=vals)
    o.setup(n=n, b=1, p=0, row_ptr=rp, col_ind=ci, vals=vals)
    assert g.nlevels == o.nlevels >= 2
    for l in range(o.nlevels):
        a, b = g.level(l), o.level(l)
        assert np.array_equal(a["row_ptr"], b["row_ptr"])
        assert np.array_equal(a["col_ind"], b["col_ind"])
        assert np.array_equal(a["val"], b["val"])
        if l + 1 < o.nlevels:
            assert np.array_equal(a["agg"], b["agg"])
    g.close()
    o.close()
