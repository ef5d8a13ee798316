"""Block triangular solves with many levels (one launch per direction) against
the oracle's factors: row by row L U z = r to 1e-13 (|L||U||z| + |r|), and the
oracle's solve to 1e-12 of its largest entry; the FP32 apply to 1e-5, as in
test_gpu_parity.py."""
import types

import numpy as np
import pytest
import torch

import _checks as K
from oracle import oracle as O
from paper_2208_08594_amd import msp, synth

pytestmark = pytest.mark.gpu


def chain(n, b):
    """Block tridiagonal: n levels of one row."""
    rng = np.random.default_rng(n)
    rp = np.concatenate([[0], np.cumsum([2] + [3] * (n - 2) + [2])]).astype(np.int32)
    ci = np.concatenate([[0, 1]] + [[i - 1, i, i + 1] for i in range(1, n - 1)] +
                        [[n - 2, n - 1]]).astype(np.int32)
    return _system(n, b, rp, ci, rng)


def box(m, b):
    """27-point box: rows of up to 13 lower entries, 8 levels in color order."""
    i = np.arange(m ** 3)
    x, y, z = i % m, i // m % m, i // (m * m)
    cols = [[] for _ in range(m ** 3)]
    for c in range(m ** 3):
        for dz in (-1, 0, 1):
            for dy in (-1, 0, 1):
                for dx in (-1, 0, 1):
                    a, e, f = x[c] + dx, y[c] + dy, z[c] + dz
                    if 0 <= a < m and 0 <= e < m and 0 <= f < m:
                        cols[c].append(a + m * (e + m * f))
    rp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    return _system(m ** 3, b, rp, np.concatenate(cols).astype(np.int32), np.random.default_rng(m))


def _system(n, b, rp, ci, rng):
    vals = rng.uniform(-1, 1, (len(ci), b, b))
    rows = np.repeat(np.arange(n), np.diff(rp))
    vals[rows == ci] += 4.0 * b * np.eye(b) * np.diff(rp)[:, None, None]
    return types.SimpleNamespace(n=n, b=b, p=0, N=n * b, nnzb=len(ci), row_ptr=rp, col_ind=ci,
                                 vals=vals, rhs=np.ones(n * b))


CASES = [
    ("chain", lambda: chain(2, 3), 0),
    ("chain", lambda: chain(300, 1), 0),
    ("chain", lambda: chain(333, 5), 0),
    ("grid", lambda: synth.lognormal_grid(24, 20, 11, 2, 3, 1.5, 0.1, "lateral4"), 0),
    ("grid", lambda: synth.lognormal_grid(9, 17, 13, 4, 3, 1.0, 1.0, "corners2"), 0),
    ("grid", lambda: synth.lognormal_grid(13, 9, 7, 6, 3, 1.0, 1.0, "corners2"), 0),
    ("grid", lambda: synth.lognormal_grid(13, 9, 7, 7, 3, 1.0, 1.0, "corners2"), 0),
    ("grid", lambda: synth.lognormal_grid(8, 8, 8, 8, 3, 1.0, 1.0, "corners2"), 0),
    ("box", lambda: box(9, 3), 1),
    ("box", lambda: box(7, 4), 0),
]


@pytest.mark.parametrize("k", range(len(CASES)))
@pytest.mark.parametrize("fp32", [False, True])
def test_sweeps(k, fp32):
    name, make, order = CASES[k]
    s = make()
    print("[case]", name, s.n, s.b, "order", order, "fp32", fp32, flush=True)
    g = msp.Solver(max_coarse=10000, bilu_order=order, precond_fp32=fp32)
    g.setup(s)
    if s.n > 2:
        assert g.info()["bilu_levels_fwd"] > 4
    o = O.OracleSolver(max_coarse=10000, bilu_order=order, precond_fp32=fp32)
    o.setup(s)
    r = np.random.default_rng(3).uniform(-1, 1, s.N)
    if fp32:
        z = g.apply(r)
        K.assert_entrywise(z.cpu().numpy(), o.apply(r), 1e-5, np.abs(o.apply(r)).max(), "apply")
        again = g.apply
    else:
        z = g.bilu_apply(r)
        F, D = o.bilu()
        perm = (O.multicolor_order(s.row_ptr, s.col_ind) if order else np.arange(s.n))
        L, U = K.bilu_factors(s, F, D, perm)
        zo = o.bilu_apply(r)
        K.bilu_backward_error(L, U, r, z.cpu().numpy(), 1e-13, "L U z = r")
        K.assert_entrywise(z.cpu().numpy(), zo, 1e-12, np.abs(zo).max(), "vs oracle")
        again = g.bilu_apply
    # a NaN or an infinity reaches the rows that depend on it and no later solve
    for bad in (np.nan, np.inf, -np.inf):
        v = r.copy()
        v[0] = bad
        w = again(v)
        assert not torch.isfinite(w).all()
        assert torch.equal(again(r), z)
    # the pending pattern itself as an input
    v = r.copy()
    v.view(np.uint64)[s.N // 2] = 0x7FF4A5A5A5A5A5A5
    assert not torch.isfinite(again(v)).all()
    assert torch.equal(again(r), z)
    g.close()
    o.close()


def test_sweeps_on_several_streams():
    """Contexts that sweep at the same time, each on its own stream."""
    ss = [synth.lognormal_grid(20, 16 + i, 12, 3, i, 1.0, 1.0, "corners2") for i in range(6)]
    gs = [msp.Solver(max_coarse=10000, bilu_order=0) for _ in ss]
    one = []
    for g, s in zip(gs, ss):
        g.setup(s)
        one.append(g.solve(s.rhs)[0])
    st = [torch.cuda.Stream() for _ in ss]
    vs = [torch.as_tensor(s.rhs, device="cuda") for s in ss]
    ref = [g.apply(v) for g, v in zip(gs, vs)]
    torch.cuda.synchronize()
    out = [[] for _ in ss]
    for rep in range(5):
        for i, g in enumerate(gs):
            with torch.cuda.stream(st[i]):
                out[i].append(g.apply(vs[i]))
    torch.cuda.synchronize()
    for i in range(len(ss)):
        assert all(torch.equal(z, ref[i]) for z in out[i])
        assert torch.equal(gs[i].solve(ss[i].rhs)[0], one[i])
        gs[i].close()
