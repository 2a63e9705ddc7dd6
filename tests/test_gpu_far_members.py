"""Explicit cells whose members lie at the very end of a member list of 2^31 - 1
entries, the longest that 32-bit offsets can address: the same masses and
counts as with the members at its beginning."""
import numpy as np
import pytest

from paper_2507_21239_amd import workloads as W

from gpu_common import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LONGEST = 2 ** 31 - 1


@pytest.mark.parametrize("max_cell", [300, 1000])   # one launch plans the first, five the second
def test_members_at_the_end_of_the_longest_list(max_cell):
    from paper_2507_21239_amd import api
    work = W.c4_batched(seed=9, counts=np.array([40, 0, 300, 77] * 40, dtype=np.int32), events=20)
    work["params"]["dm_max"] = 1e-3
    n = len(work["particles"]["m"])
    order = torch.empty(LONGEST, dtype=torch.int32, device="cuda")
    got = []
    for at in (0, LONGEST - n):
        say("members at", at, "max_cell", max_cell)
        cells = api.cells_to_device(work["cells"])
        order[at:at + n] = cells["order"]
        far = dict(cells, cell_start=cells["cell_start"] + at, order=order)
        dev = api.to_device(work["particles"])
        counts = api.collide_noalloc(work["params"], dev, far, 0.0, 20, step=1, max_cell=max_cell)
        counts, m = counts.cpu().numpy(), dev["m"].cpu().numpy()
        dev = api.to_device(work["particles"])
        sim = api.Simulation(work["params"], dev)
        sim.bin(far, max_cell=max_cell)
        sim.step(0.0, 20, 2)
        st = sim.stats()
        sim.close()
        got.append((counts, m, st["events"], dev["m"].cpu().numpy()))
        assert counts[5] == 0 and st["device_flags"] == 0 and st["events"] > 0
    for a, b in zip(*got):
        assert np.array_equal(a, b)
