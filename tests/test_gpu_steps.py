"""The scalar steps of the plug-in rule and the bandwidth grid run at the end of
the kernel before them where a pass's lists name the same columns (a call), and
in launches of their own where they differ: columns of two and three stages,
of the selectors' subsets, and with stages that fail, together in one batch.
Both routes run the same device code, so a column's plug-in results are the
same bit for bit; g sums the same FP32 runs in FP64 in another grouping (at
most 2^15 partial sums of one sign: 2^15 x 2^-53 = 3.6e-12 of gscale)."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _requests(kde):
    R, P, L = kde.KDE_METHOD_ROT, kde.KDE_METHOD_PLUGIN, kde.KDE_METHOD_LSCV
    grid = ("log_rot", 0.1, 2.0, 40)
    out = []
    for k, (methods, stages, n, dtype) in enumerate([
            (R | P | L, 3, 1500, np.float32), (R | P | L, 2, 700, np.float64), (R | L, 3, 900, np.float32),
            (R | P, 2, 2600, np.float32), (R, 3, 300, np.float64), (R | P | L, 3, 513, np.float64)]):
        out.append(kde.Request(workloads.draw("bimodal", n, 60 + k, dtype), methods, stages, grid))
    out.append(kde.Request(np.full(400, 2.5, np.float32), R | P | L, 3, grid))  # zero spread
    return out


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("kappa", [0, 1, 1000])
def test_steps_of_mixed_batches_are_those_of_single_columns(precision, kappa):
    import paper_1505_01998_amd as kde

    reqs = _requests(kde)
    with kde.Context(0, precision) as c:
        c.set_option("fp64_kappa", kappa)
        batch = c.batch(reqs)
        alone = [c.batch([r])[0] for r in reqs]
    assert batch[-1].status == alone[-1].status == kde.KDE_E_DEGENERATE
    for r, a, b in list(zip(reqs, alone, batch))[:-1]:
        assert a.status == b.status == kde.KDE_OK
        assert a.sigma == b.sigma and a.h_rot == b.h_rot
        if r.methods & kde.KDE_METHOD_PLUGIN:
            assert a.h_plugin == b.h_plugin > 0
            assert np.array_equal(a.plugin.psi, b.plugin.psi)
            assert np.array_equal(a.plugin.g, b.plugin.g, equal_nan=True)  # NaN: no such stage
        if r.methods & kde.KDE_METHOD_LSCV:
            assert a.k_lscv == b.k_lscv
            assert np.all(np.abs(a.g - b.g) <= 2.0**-38 * a.gscale)


@pytest.mark.parametrize("n", [2, 255, 257, 2047, 2048])
def test_moments_of_small_columns_do_not_depend_on_the_batch(n):
    """One launch where every column of a call has at most 2048 samples, four
    beside a longer one: the same sums, bit for bit; a column that holds a
    non-finite value is refused by both."""
    import paper_1505_01998_amd as kde

    x, bad = workloads.draw("lognormal", n, 90 + n, np.float64), np.arange(n, dtype=np.float64)
    bad[n // 2] = np.inf
    rot = [kde.Request(v, kde.KDE_METHOD_ROT, 3, ("paper", 8)) for v in (x, bad)]
    long = kde.Request(workloads.draw("gamma", 5000, 91, np.float32), kde.KDE_METHOD_ROT, 3, ("paper", 8))
    with kde.Context(0) as c:
        alone, beside = c.batch(rot), c.batch(rot + [long])
    assert alone[0].status == beside[0].status == kde.KDE_OK
    assert alone[0].sigma == beside[0].sigma and alone[0].h_rot == beside[0].h_rot
    want = float(np.std(x, ddof=1))
    assert abs(alone[0].sigma - want) <= (n + 10) * 2.0**-53 * want
    assert alone[1].status == beside[1].status == kde.KDE_E_INVAL
