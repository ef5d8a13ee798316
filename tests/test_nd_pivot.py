"""The pivots' reciprocals of the nested-dissection coarsest solver: those of an
IEEE division, also for the mantissas just below a power of two, where Newton
steps on an estimate end one unit in the last place off."""
import numpy as np
import pytest

from paper_2208_08594_amd import msp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_reciprocal_is_rounded_once(sign):
    """Pairs [[1, b], [a, 1]] with a b = k 2^-53 exactly: the second pivot is
    1 - a b and the solve for (0, 1) returns its reciprocal."""
    k = np.arange(1, 1025, dtype=np.float64)
    n = 2 * k.size
    rp = np.arange(0, 2 * n + 1, 2, dtype=np.int32)
    ci = np.repeat(np.arange(n) // 2 * 2, 2).astype(np.int32) + np.tile([0, 1], n).astype(np.int32)
    vals = np.ones((k.size, 2, 2))
    vals[:, 0, 1] = sign * 2.0 ** -23
    vals[:, 1, 0] = sign * k * 2.0 ** -30
    g = msp.Solver(max_coarse=10000)
    g.setup(n=n, b=1, p=0, row_ptr=rp, col_ind=ci, vals=vals.reshape(-1, 1, 1))
    assert g.nlevels == 1
    A = g.level(0)
    assert np.array_equal(A["val"], vals.reshape(-1))  # unit diagonal: nothing to decouple
    f = np.tile([0.0, 1.0], k.size)
    x = g.vcycle(f).cpu().numpy()[1::2]
    assert np.array_equal(x, 1.0 / (1.0 - k * 2.0 ** -53))
    g.close()
