"""Range aggregates at the edges of their kernel: columns around a wave and a
block, ranges that no sample, one end or both ends of a kernel reach, ranges
so far out that only the pass over every sample keeps their digits, empty and
infinite ones, and bandwidths from far below the samples' spacing to far above
their range.  A sample's share is an exact function of two standardised
distances z; rounding z (2^-53) moves a tail Q(z) by about z^2 2^-53 of itself
and the exponential and the polynomial add a few 2^-53, so COUNT is held to
1e-12 of itself for |z| <= 38 (1444 x 2 x 1.1e-16 = 3.2e-13), SUM to 1e-12 of
COUNT times the largest |x| + 40 h.  The reference takes each share between
tails from scipy's normal distribution function (the oracle's differences of
the distribution function keep no digits of an upper tail)."""
import numpy as np
import pytest
from scipy.special import ndtr

import workloads

pytestmark = pytest.mark.gpu


def _reference(x, h, lo, hi):
    x = x.astype(np.float64)
    cnt, sm = np.zeros(len(lo)), np.zeros(len(lo))
    for k, (a, b) in enumerate(zip(lo, hi)):
        al, be = (a - x) / h, (b - x) / h
        p = np.where(al >= 0, ndtr(-al) - ndtr(-be), np.where(be <= 0, ndtr(be) - ndtr(al), 1 - ndtr(al) - ndtr(-be)))
        d = (np.exp(-0.5 * al * al) - np.exp(-0.5 * be * be)) / np.sqrt(2 * np.pi)
        cnt[k], sm[k] = p.sum(), (x * p + h * d).sum()
    return cnt, sm


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 257, 4097])
@pytest.mark.parametrize("scale", [1e-4, 0.05, 3.0, 1e3])
def test_ranges_at_the_edges(n, dtype, scale):
    import paper_1505_01998_amd as kde

    x = workloads.draw("bimodal", n, 900 + n, dtype)
    xs = np.sort(x.astype(np.float64))
    h = scale * 0.7
    mid = float(xs[n // 2])
    lo = [-np.inf, -np.inf, mid, mid, mid - 1e-3 * h, xs[0] - 30 * h, xs[-1] + 5 * h, xs[-1] + 20 * h, mid + 8.9 * h,
          xs[0] - 13 * h, xs[0], np.inf, mid - 40 * h]
    hi = [np.inf, mid, np.inf, mid, mid + 1e-3 * h, xs[0] - 25 * h, xs[-1] + 6 * h, np.inf, mid + 12.1 * h,
          xs[0] - 11 * h, xs[-1], np.inf, mid + 40 * h]
    lo, hi = np.array(lo), np.array(hi)
    oc, osm = _reference(x, h, lo, hi)
    with kde.Context(0) as c:
        cnt, sm, avg = c.range_aggregates(x, h, lo, hi)
        again = c.range_aggregates(x, h, lo[::-1].copy(), hi[::-1].copy())
    far = float(np.abs(xs).max()) + 40 * h
    assert np.all(np.abs(cnt - oc) <= 1e-12 * oc + 1e-300)
    assert np.all(np.abs(sm - osm) <= 1e-12 * oc * far + 1e-300)
    assert cnt[3] == 0.0 and np.isnan(avg[3]) and cnt[11] == 0.0
    # a range's result does not depend on the others of the call
    assert np.array_equal(again[0][::-1], cnt) and np.array_equal(again[1][::-1], sm)
