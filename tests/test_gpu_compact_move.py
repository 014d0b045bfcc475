"""Exit nodes on few rows: the partition and the moves of the rows that go on
are one launch up to 1024 rows and 128 KB (128 rows of the MLP's 256 floats),
two above.  A row's results do not depend on the batch it came in, so each
batch gives the first rows of a batch of 300, bit for bit, in all host modes;
its branch counts add up; and the oracle agrees (test_gpu_host_modes).  A
network of narrow layers takes one launch up to the 1024 rows themselves, with
two tensors moved at once."""

import json

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


def _narrow_plan():
    """Two hidden layers of 16 floats, both carried past the first exit (8
    vectors of 16 bytes a row: 1024 rows are the 128 KB), the second one past the
    next exit too; the third layer reads it there."""
    from paper_2307_04963_amd import runtime
    rng = np.random.default_rng(5)
    blob = bytearray()

    def add(arr):
        blob.extend(b"\0" * ((-len(blob)) % 256))
        at = len(blob)
        blob.extend(np.asarray(arr, np.float32).tobytes())
        return at

    def linear(src, dst, cin, cout):
        return {"op": "conv", "src": src, "dst": dst, "k": 1, "cout": cout, "act": "relu",
                "w": {"off": add(rng.uniform(-1, 1, (cout, cin)))}, "shift": add(rng.uniform(-0.2, 0.2, cout))}

    def head(src, index, **more):
        return {"op": "exit", "src": src, "w": add(rng.uniform(-1, 1, (10, 16))), "b": add(rng.uniform(-1, 1, 10)),
                "T": add([1.0]), "ncls": 10, "index": index, "final": index == 2, **more}

    spec = {"version": 1, "dtype": "f32", "input": {"name": "x", "shape": [8]}, "n_out": 10,
            "nodes": [linear("x", "a", 8, 16), linear("x", "b", 8, 16),
                      head("a", 0, tau=0.6, carry=[["a", "ac"], ["b", "bc"]]),
                      linear("ac", "c", 16, 16), head("c", 1, tau=0.6, carry=[["bc", "bd"]]),
                      linear("bd", "d", 16, 16), head("d", 2)]}
    return runtime.Plan(json.dumps(spec), bytes(blob), 1100)


@pytest.mark.parametrize("mode", ["sync", "device", "graph"])
def test_exit_up_to_1024_rows(mode):
    import torch
    plan = _narrow_plan()
    x = torch.from_numpy(np.random.default_rng(6).standard_normal((1100, 8)).astype(np.float32)).cuda()

    def run(n):
        logits, rec, _ = plan.outputs(n)
        plan.run(x[:n], None, logits, rec)
        torch.cuda.synchronize()
        return logits, rec, plan.counts()

    logits, rec, counts = run(1100)      # more than 1024 rows: partition and moves in two launches
    assert all(100 < c[0] < 900 for c in counts), counts
    plan.set_host_mode(mode)
    for n in (1, 129, 513, 1000, 1023, 1024, 1025):
        for _ in range(2):               # the second run knows the first one's counts
            got, grec, gcounts = run(n)
            assert torch.equal(got, logits[:n]) and torch.equal(grec, rec[:n])
            rows = n
            for taken, left in gcounts:
                assert taken + left == rows
                rows = left
            assert rows == 0
    plan.close()
