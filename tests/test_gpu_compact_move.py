"""Exit nodes on few rows: the partition and the moves of the rows that go on
are one launch up to 1024 rows and 128 KB (128 rows of the MLP's 256 floats),
two above.  A row's results do not depend on the batch it came in, so each
batch gives the first rows of a batch of 300, bit for bit, in all host modes;
its branch counts add up; and the oracle agrees (test_gpu_host_modes)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

_whole = {}


def _plan():
    from paper_2307_04963_amd import runtime
    from workloads import configs
    if not _whole:
        wl = configs.build("mlp_exit")
        plan = runtime.Plan.from_workload(wl, 300)
        x, aux = wl.inputs(300)
        _whole.update(wl=wl, plan=plan, x=x, rt=runtime, ref=runtime.run_numpy(plan, wl, x, aux))
    return _whole


@pytest.mark.parametrize("mode", ["sync", "device", "graph"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 300])
def test_exit_few_rows(n, mode):
    s = _plan()
    s["plan"].set_host_mode(mode)
    try:
        for _ in range(2):   # the second run knows the first one's counts
            got = s["rt"].run_numpy(s["plan"], s["wl"], s["x"][:n])
    finally:
        s["plan"].set_host_mode("sync")
    assert np.array_equal(got["logits"], s["ref"]["logits"][:n])
    assert np.array_equal(got["exit_index"], s["ref"]["exit_index"][:n])
    rows = n
    for taken, left in got["counts"]:
        assert taken + left == rows
        rows = left
    assert rows == 0
