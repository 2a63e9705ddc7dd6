"""The batched kernels' event loops compiled for a fixed number of slots per
lane (1 to 4) and for one event budget, against the loop with the number of
slots and the budget read at run time.

The plain schedule runs every cell on a four-wave team through the loop that
reads both; the batched schedule with a single-wave threshold of 0 runs the
same teams through the specialised loops.  Same layout, same operations in the
same order: masses, compositions and counters must be equal bit for bit.  The
cells' sizes are the edges of the slot counts and of the waves within a team."""
import numpy as np
import pytest

from paper_2507_21239_amd import workloads as W

from gpu_common import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [1, 2, 63, 64, 65, 192, 193, 255, 256, 257, 300, 511, 512, 513, 767, 768, 769, 1023, 1024]


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("comp", [0, 3])
@pytest.mark.parametrize("limit", ["count", "time"])
def test_specialised_loops_equal_the_general_one(precision, comp, limit):
    from paper_2507_21239_amd import api
    work = W.c4_batched(seed=17, counts=SIZES, events=70, philox_seed=5)
    work["params"]["n_comp"] = comp
    if comp:
        rng = np.random.default_rng(2)
        c = rng.random((comp, len(work["particles"]["m"])))
        work["particles"]["comp"] = (c / c.sum(axis=0)).astype(np.float32)
    # 1e7 s: from no event to a few hundred, over the batches of 64 uniforms
    dt, count = (0.0, 70) if limit == "count" else (1.0e7, 0)
    got = []
    for schedule in ("plain", "batched"):
        say("event loops", precision, "comp", comp, limit, schedule)
        dev = api.to_device(work["particles"])
        sim = api.Simulation(work["params"], dev, precision=precision, schedule=schedule)
        sim.bin(api.cells_to_device(work["cells"]))
        if schedule == "batched":
            sim.set_schedule(0, 0)
        sim.step(dt, count, 1)
        st = sim.stats()
        got.append((st, {k: dev[k].cpu().numpy() for k in ("m", "comp") if k in dev}))
        sim.close()
    (sa, a), (sb, b) = got
    assert sa["events"] == sb["events"] > len(SIZES)
    assert sa["outcomes"] == sb["outcomes"]
    for k in a:
        assert np.array_equal(a[k], b[k]), k
