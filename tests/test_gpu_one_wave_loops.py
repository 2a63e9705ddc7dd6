"""The one-wave event loops at the edges of their slot counts (1 to 4 a lane),
for both event budgets, with and without fractions and event log: FP64 against
the oracle's event log and masses, and in both precisions the kernels with the
event log compiled in against those without, bit for bit."""
import numpy as np
import pytest

from paper_2507_21239_amd import workloads as W

from gpu_common import compare_logs, run_gpu_explicit, run_oracle_explicit, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256]
EVENTS = 130    # two batches of uniforms and a part


def _work(limit, comp):
    work = W.c4_batched(seed=31, counts=SIZES, events=EVENTS, philox_seed=7)
    work["params"]["n_comp"] = comp
    if comp:
        c = np.random.default_rng(2).random((comp, len(work["particles"]["m"])))
        work["particles"]["comp"] = (c / c.sum(axis=0)).astype(np.float32)
    if limit == "time":
        work.update(dt=1.0e7, max_events=0)   # from no event to a few hundred
    return work


@pytest.mark.parametrize("comp", [0, 3])
@pytest.mark.parametrize("limit", ["count", "time"])
def test_fp64_one_wave_loops_follow_the_oracle(limit, comp):
    work = _work(limit, comp)
    opart, oout = run_oracle_explicit(work, log_per_cell=600)
    assert int(oout["stats"]["events"].max()) < 600 and int(oout["stats"]["events"].sum()) > 200
    gpart, gstats, glog = run_gpu_explicit(work, "fp64", "batched", log_per_cell=600)
    assert compare_logs(oout["log"], oout["stats"], glog) == []
    assert gstats["device_flags"] == 0
    ok = np.abs(gpart["m"] - opart["m"]) <= 1e-12 * opart["m"]
    assert ok.all()


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("frag", ["sharp", "maxwell"])
@pytest.mark.parametrize("limit", ["count", "time"])
def test_kernels_with_and_without_the_log_agree(precision, frag, limit):
    work = _work(limit, 0)
    work["params"]["frag_mode"] = frag
    say("log or not", precision, frag, limit)
    a, sa, _ = run_gpu_explicit(work, precision, "batched")
    b, sb, _ = run_gpu_explicit(work, precision, "batched", log_per_cell=4)
    assert sa == sb and sa["events"] > 200
    assert np.array_equal(a["m"], b["m"])
