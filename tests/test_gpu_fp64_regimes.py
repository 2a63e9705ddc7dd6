"""FP64 pair rates over all Stokes regimes of the turbulent velocity (both
particles coupled, one, none) and grouping factors from off to nearly one,
against the oracle, row-normwise.  Bound 1e-13 as for the FP64 rates of the
parity tests: about ten roundings of a rate and the row sum's, with the
cancellation of near-identical particles weighed by their share of the row."""
import numpy as np
import pytest

import oracle as O
from paper_2507_21239_amd import workloads as W

from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dm_max", [0.0, 1e-3, 0.9])
@pytest.mark.parametrize("lo,hi", [(-12.0, -6.0), (-12.0, 8.0), (4.0, 9.0)])
def test_fp64_rates_over_the_stokes_regimes(dm_max, lo, hi):
    from paper_2507_21239_amd import api
    say("fp64 regimes", dm_max, lo, hi)
    counts = [2, 65, 257]
    work = W.c4_batched(seed=9, counts=counts, events=1)
    work["params"]["dm_max"] = dm_max
    part = work["particles"]
    part["m"][:] = 10.0 ** np.random.default_rng(10).uniform(lo, hi, len(part["m"]))
    part["m"][1::7] = part["m"][::7][:len(part["m"][1::7])]  # equal masses
    sim = api.Simulation(work["params"], api.to_device(part), precision="fp64")
    sim.bin(api.cells_to_device(work["cells"]))
    cs = work["cells"]["cell_start"]
    for c, n in enumerate(counts):
        got, sums = (x.cpu().numpy() for x in sim.rates(c, n))
        ref, rsum = O.cell_rates(work["params"], work["cells"]["gas"][c],
                                 work["cells"]["order"][cs[c]:cs[c + 1]], part["m"], part["M"])
        assert np.max(np.abs(got - ref) / rsum[:, None]) <= 1e-13, (c, n)
        assert np.max(np.abs(sums - rsum) / rsum) <= 1e-13, (c, n)
    sim.close()
