"""FP64 starting row sums at the lines between their forms -- one-wave cells of up
to 32 lanes, which end after their last pair of lanes; four-wave teams of up to
192 members, which sum every row over the members; larger teams with waves that
hold no particle -- against the oracle: 1e-13 relative, as for the FP64 row sums
in general.  The events that follow must equal the oracle's one for one."""
import numpy as np
import pytest

import oracle as O
from paper_2507_21239_amd import workloads as W

from gpu_common import compare_logs, run_gpu_explicit, run_oracle_explicit, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [1, 2, 3, 30, 31, 32, 33, 34, 64, 65, 66, 128, 129, 191, 192, 193, 194, 256, 257, 258, 320,
         321, 384, 385, 512, 513, 576, 577, 768, 769]


@pytest.mark.parametrize("schedule,small_max", [("batched", 256), ("batched", 0), ("plain", None)])
@pytest.mark.parametrize("kernel", ["physical", "constant"])
def test_fp64_rows_at_the_lines_between_their_forms(schedule, small_max, kernel):
    from paper_2507_21239_amd import api
    work = W.c4_batched(seed=21, counts=SIZES, events=25, philox_seed=3)
    work["params"]["kernel"] = kernel
    cells, part = work["cells"], work["particles"]
    say("row forms", schedule, small_max, kernel)
    sim = api.Simulation(work["params"], api.to_device(part), precision="fp64", schedule=schedule)
    sim.bin(api.cells_to_device(cells), max_cell=max(SIZES))
    if small_max is not None:
        sim.set_schedule(small_max, 0)
    got = sim.row_sums(len(part["m"])).cpu().numpy()
    sim.close()
    for c in range(len(SIZES)):
        s = slice(int(cells["cell_start"][c]), int(cells["cell_start"][c + 1]))
        _, rows = O.cell_rates(work["params"], cells["gas"][c], cells["order"][s], part["m"], part["M"])
        ok = np.abs(got[s] - rows) <= 1e-13 * np.abs(rows)
        assert ok.all(), SIZES[c]
    opart, oout = run_oracle_explicit(work, log_per_cell=25)
    gpart, gstats, glog = run_gpu_explicit(work, "fp64", schedule, log_per_cell=25,
                                           batched_schedule=None if small_max is None else (small_max, 0))
    assert compare_logs(oout["log"], oout["stats"], glog) == []
    assert gstats["device_flags"] == 0
