"""Null events (tests/test_oracle_null_event.py) are no anomaly: they form no
new mass, so no device flag may rise from them, whatever the grouping of
collisions.  400 of that test's three-particle cells with swarm masses of their
own, so that many of them end in null events.  Their mass ratio is 16 and the
grouping factor 1 with dm_max = 1e-3 as with 0; masses and the real events must
equal the oracle's."""
import numpy as np
import pytest

from gpu_common import run_gpu_explicit, run_oracle_explicit, say
from test_oracle_null_event import null_event_work

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CELLS = 400


def _work(dm_max):
    work = null_event_work(1)
    work["params"]["dm_max"] = dm_max
    part, c = work["particles"], work["cells"]
    M = np.random.default_rng(8).uniform(0.2, 7.0, 3 * CELLS)
    work["particles"] = dict(r=np.zeros(3 * CELLS), z=np.zeros(3 * CELLS), m=np.tile(part["m"], CELLS),
                             M=M, active=np.ones(3 * CELLS, dtype=np.uint8), comp=None)
    work["cells"] = dict(cell_start=np.arange(0, 3 * CELLS + 1, 3, dtype=np.int32),
                         order=np.arange(3 * CELLS, dtype=np.int32), gas=np.tile(c["gas"], (CELLS, 1)))
    return work


@pytest.mark.parametrize("dm_max", [0.0, 1e-3])
@pytest.mark.parametrize("schedule,small_max", [("plain", None), ("batched", 256), ("batched", 0)])
def test_null_events_raise_no_flag(schedule, small_max, dm_max):
    work = _work(dm_max)
    opart, oout = run_oracle_explicit(work, log_per_cell=60)
    gpart, gstats, glog = run_gpu_explicit(work, "fp64", schedule, log_per_cell=60,
                                           batched_schedule=None if small_max is None else (small_max, 0))
    nulls = 0
    for c in range(CELLS):
        o = np.stack([oout["log"][c][k][:int(oout["stats"]["events"][c])]
                      for k in ("i", "j", "outcome")], axis=1)
        g = glog[c][glog[c][:, 0] != -7, :3]
        assert np.array_equal(g[g[:, 1] >= 0], o[o[:, 1] >= 0]), c
        nulls += int(np.sum(g[:, 1] < 0))
    say("null events", nulls)
    assert nulls > 0
    assert np.array_equal(gpart["m"], opart["m"])
    assert gstats["device_flags"] == 0 and gstats["status"] == 0


def test_null_events_of_the_context_free_call_raise_no_flag():
    from paper_2507_21239_amd import api
    work = _work(1e-3)
    say("null events, context-free")
    opart, oout = run_oracle_explicit(work)
    dev = api.to_device(work["particles"])
    counts = api.collide_noalloc(work["params"], dev, api.cells_to_device(work["cells"]), 0.0,
                                 work["max_events"], step=0, precision="fp64", max_cell=3).cpu().numpy()
    real = int(counts[1:5].sum())
    assert real == int(oout["stats"]["outcomes"].sum()) and counts[0] > real
    assert counts[5] == 0
    assert np.array_equal(dev["m"].cpu().numpy(), opart["m"])
