"""Range ends that coincide with samples at zero, where a standardised distance
is a zero of either sign: ends of -0.0, both zeros as the two ends of an empty
range, and samples so close to an end that the distance over h underflows.
COUNT is held to 1e-12 of itself, as in test_gpu_ranges.py, and SUM to 1e-12 of
COUNT times the largest |x| + 40 h; the normal distribution function is exactly
1/2 at both zeros."""
import numpy as np
import pytest
from scipy.special import ndtr

pytestmark = pytest.mark.gpu

_TINY = 5e-324  # the smallest subnormal


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("h", [0.25, 4.0])
@pytest.mark.parametrize("n", [3, 64, 1000])
def test_ranges_that_end_at_zero(n, h, dtype):
    import paper_1505_01998_amd as kde

    x = np.zeros(n, dtype)
    x[::3] = np.random.default_rng(n).normal(0.0, 2.0, x[::3].size)
    x[1::3] = -0.0
    lo = np.array([-0.0, 0.0, -np.inf, -np.inf, -0.0, 0.0, -1.0, -0.0])
    hi = np.array([np.inf, np.inf, -0.0, 0.0, 1.0, 1.0, -0.0, 0.0])
    lo, hi = np.append(lo, 0.0), np.append(hi, -0.0)
    x64 = x.astype(np.float64)
    with kde.Context(0) as c:
        cnt, sm, _ = c.range_aggregates(x, h, lo, hi)
    far = float(np.abs(x64).max()) + 40 * h
    for k in range(len(lo)):
        al, be = (lo[k] - x64) / h, (hi[k] - x64) / h
        want = (ndtr(be) - ndtr(al)).sum()
        ends = [np.exp(-0.5 * z * z) / np.sqrt(2 * np.pi) for z in (al, be)]
        want_sum = (x64 * (ndtr(be) - ndtr(al)) + h * (ends[0] - ends[1])).sum()
        assert abs(cnt[k] - want) <= 1e-12 * n, (k, lo[k], hi[k])
        assert abs(sm[k] - want_sum) <= 1e-12 * n * far, (k, lo[k], hi[k])
    assert cnt[-2] == 0.0 and cnt[-1] == 0.0


@pytest.mark.parametrize("tiny,h", [(_TINY, 4.0), (1e-310, 1e20), (_TINY, 1e-3)])
def test_ranges_of_samples_next_to_an_end(tiny, h):
    """Half of each sample's kernel lies on either side of an end that the
    sample all but touches, above it or below."""
    import paper_1505_01998_amd as kde

    x = np.array([tiny, -tiny])
    lo, hi = np.array([0.0, -np.inf, -0.0]), np.array([np.inf, 0.0, np.inf])
    with kde.Context(0) as c:
        cnt = c.range_aggregates(x, h, lo, hi)[0]
    # the kernel's density at the end is below 400 and the distance below 1e-306
    assert np.allclose(cnt, 1.0, rtol=1e-12, atol=0)
