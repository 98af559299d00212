"""The range kernel passes samples between the lanes of a wave through a queue
in LDS.  A wave's LDS operations execute in program order, so no instruction is
needed between them, but the compiler has to be told that they depend on each
other across lanes: in the assembly of the pass with the queue a scheduling
barrier stands between the store and the loads that follow it, and between the
load in the loop and the next round's store.  The source is compiled to
assembly here; no GPU is needed."""
import os
import re
import subprocess

import pytest

from paper_1505_01998_amd import build as b


@pytest.mark.skipif(not os.path.exists(b.hipcc()), reason="hipcc missing")
def test_range_queue_is_ordered_across_lanes(tmp_path):
    out = tmp_path / "query.s"
    subprocess.run([b.hipcc(), *b.HIPCC_FLAGS, "-I", os.path.join(b.ROOT, "include"), "-I", b.CSRC,
                    "--offload-device-only", "-S", "-o", str(out), os.path.join(b.CSRC, "kde_query.hip")],
                   check=True, capture_output=True)
    m = re.search(r"^\S*k_range_f64ILb0\S*:.*?\n(.*?)\.Lfunc_end", out.read_text(), re.M | re.S)
    assert m
    # up to the first block barrier, behind which the sums of the block follow
    ops = re.findall(r"; wave barrier|\bds_write_b64|\bds_read_b64|\bs_barrier", m.group(1))
    ops = ops[:ops.index("s_barrier")]
    stores = [k for k, o in enumerate(ops) if o == "ds_write_b64"]
    # the queue's store, its load in the loop and the one after it; the last
    # store starts the block's sums
    assert len(stores) == 2 and ops.count("ds_read_b64") == 2
    queue = ops[stores[0]:stores[1]]
    assert queue == ["ds_write_b64", "; wave barrier", "ds_read_b64", "; wave barrier", "ds_read_b64"]
