"""The FP64 sweep's exponential, one pair at a time: two samples a distance 1
apart, so S1(h) is e^-x with x = 1 / (4 h^2) and S2(h) its square.  x is formed
with about three roundings (2^-53 of x each), the exponential is within 1.02
2^-53 and the square adds one: S1 is held to (2 + 3 x) 2^-53 of itself, S2 to
twice that and one more.  Every residue of the 64-entry table and both ends of
its intervals occur, and x beyond 746 gives exactly 0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("part", range(4))
def test_fp64_sweep_of_one_pair(part):
    import paper_1505_01998_amd as kde

    step = np.log(2.0) / 64
    k = np.arange(part, 64 * 1000, 251, dtype=np.float64)  # 251 and 64 are coprime
    x = np.concatenate([[1e-12], (k + 0.499) * step, (k + 0.501) * step, [746.0, 1e3, 1e7, 1e300]])
    x = -np.unique(-x)  # the grid ascends
    h = 0.5 / np.sqrt(x)
    with kde.Context(0, "fp64") as c:
        s1, s2 = c.lscv_sums(np.array([0.0, 1.0]), h)
    want = np.exp(-0.25 / h.astype(np.longdouble) ** 2)
    ok = x < 700
    assert np.all(np.abs(s1[ok] - want[ok]) <= (2 + 3 * x[ok]) * 2.0**-53 * want[ok])
    sq = x < 350
    assert np.all(np.abs(s2[sq] - want[sq] ** 2) <= (5 + 6 * x[sq]) * 2.0**-53 * want[sq] ** 2)
    assert np.all(s1[x >= 746.0] == 0.0) and np.all(s2[x >= 400.0] == 0.0)
