"""A batch of many small columns sweeps whole work items, a block running the
item's pieces one after the other; alone, a column's pieces are blocks of their
own.  Every partial sum has its slot either way, so a column's results are the
same bit for bit, in the mixed form (each number of bandwidths a block, on the
matrix cores, in the persistent launch) and in FP64.  The columns lie around
one run (64), one row (256) and one tile (512), so that items have pieces
beyond the last sample."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

_SIZES = (2, 63, 65, 200, 256, 257, 300, 511, 512, 513, 700, 1000, 1025)


@pytest.mark.parametrize("precision,options", [
    ("mixed", {}), ("mixed", {"lscv_hc": 8}), ("mixed", {"lscv_hc": 32}), ("mixed", {"lscv_mfma": 1}),
    ("mixed", {"launch_evals": 10**6}), ("mixed", {"launch_evals": 10**6, "lscv_tj": 1024}), ("fp64", {})])
def test_columns_of_a_large_batch_are_those_alone(precision, options):
    import paper_1505_01998_amd as kde

    # 1800 (of 32 bandwidths) to 6700 (of 8) whole units; from 1024 on (FP64:
    # 4096), with over 6144 pieces, they run whole
    reqs = [kde.Request(workloads.draw("bimodal", n, 7 * n + k, np.float32), kde.KDE_METHOD_LSCV, 2,
                        ("log_rot", 0.1, 2.0, 60 + 13 * k)) for k in range(12) for n in _SIZES]
    with kde.Context(0, precision) as c:
        for key, value in options.items():
            c.set_option(key, value)
        batch = c.batch(reqs)
        alone = [c.batch([r])[0] for r in reqs]
    for r, a, b in zip(reqs, alone, batch):
        assert a.status == b.status == kde.KDE_OK
        assert np.array_equal(a.g, b.g) and np.array_equal(a.gscale, b.gscale), (r.x.size, len(b.g))


def test_served_small_columns_are_those_alone():
    import paper_1505_01998_amd as kde

    reqs = [kde.Request(workloads.draw("gamma", n, 900 + k, np.float32), kde.KDE_METHOD_LSCV, 2,
                        ("log_rot", 0.1, 2.0, 100)) for k, n in enumerate(_SIZES * 12)]
    with kde.Context(0) as alone, kde.Context(0) as srv:
        want = [alone.batch([r])[0] for r in reqs]
        srv.server_start(1 << 30, 128)
        tickets = [srv.submit(r) for r in reqs]
        got = [srv.wait(t) for t in tickets]
        srv.server_stop()
    for a, b in zip(want, got):
        assert a.status == b.status == kde.KDE_OK and np.array_equal(a.g, b.g)
