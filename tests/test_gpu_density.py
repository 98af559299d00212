"""The density of few points, where sixteen waves share a block's samples,
against the kernel that many points take: both fold the same runs in the same
order over the same pieces of the column (four of 4096 samples or more here,
whatever the number of points), so a point's value is the same bit for bit.
The FP64 form, whose pieces follow the number of points, is held to the direct
sum: n roundings of the additions and 200 of a term's argument and exponential
(arguments up to 40 matter), in 2^-53."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

# a call of this many points fills the chip with 256-point blocks
_MANY = 256 * 800


@pytest.mark.parametrize("n", [16384, 16385, 16896, 17409, 20011])
@pytest.mark.parametrize("h", [1e-3, 0.3])
def test_density_of_few_points_is_that_of_many(n, h):
    import paper_1505_01998_amd as kde

    x = workloads.draw("bimodal", n, 40 + n, np.float32)
    pts = np.random.default_rng(n).uniform(x.min() - 1, x.max() + 1, _MANY)
    with kde.Context(0) as c:
        many = c.density(x, h, pts)
        for m in (1, 63, 64, 65, 300):
            assert np.array_equal(c.density(x, h, pts[:m]), many[:m]), m


@pytest.mark.parametrize("n", [2, 511, 513, 1025, 4097])
def test_density_fp64_of_few_points(n):
    import paper_1505_01998_amd as kde

    x = workloads.draw("bimodal", n, 70 + n, np.float64)
    pts, h = x[:: max(1, n // 5)][:5].copy(), 0.2
    want = np.array([np.exp(-0.5 * ((p - x) / h) ** 2).sum() for p in pts]) / (n * h * np.sqrt(2 * np.pi))
    with kde.Context(0, "fp64") as c:
        np.testing.assert_allclose(c.density(x, h, pts), want, rtol=(n + 200) * 2.0**-53)
