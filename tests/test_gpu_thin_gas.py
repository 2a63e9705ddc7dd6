"""FP64 pair rates in gas so thin that products of two Stokes numbers overflow,
down to a vacuum, where they are infinite and turbulence moves nothing: the
oracle takes each particle's 1 / (1 + St) by itself.  Bound 1e-13, as for the
FP64 rates in general."""
import numpy as np
import pytest

import oracle as O
from paper_2507_21239_amd import workloads as W

from gpu_common import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sources", [["turb"], ["brownian", "turb"]])
@pytest.mark.parametrize("rho", [1e-40, 1e-165, 1e-200, 1e-290, 0.0])
def test_fp64_rates_in_thin_gas(rho, sources):
    from paper_2507_21239_amd import api
    say("thin gas", rho, sources)
    n = 70
    p = W.benchmark_params(flags=sources + ["coag"])
    m0 = 4.0 / 3.0 * np.pi * p["a_mono"] ** 3 * p["rho_s"]
    m = m0 * 10.0 ** np.random.default_rng(3).uniform(0.0, 14.0, n)
    part = dict(r=np.zeros(n), z=np.zeros(n), m=m, M=np.ones(n), active=np.ones(n, dtype=np.uint8))
    cells = dict(cell_start=np.array([0, n], dtype=np.int32), order=np.arange(n, dtype=np.int32),
                 gas=np.array([[1e30, rho, 100.0, 1e-3, 5 * W.AU, 1.0]]))
    ref, rows = O.cell_rates(p, cells["gas"][0], cells["order"], m, part["M"])
    assert np.all(np.isfinite(ref)) and np.all(rows > 0.0) == (rho > 0.0 or "brownian" in sources)
    sim = api.Simulation(p, api.to_device(part), precision="fp64")
    sim.bin(api.cells_to_device(cells))
    got = sim.rates(0, n)[0].cpu().numpy()
    got_rows = sim.row_sums(n).cpu().numpy()
    sim.step(0.0, 5, 1)
    st = sim.stats(check=False)
    sim.close()
    ok = np.abs(got - ref) <= 1e-13 * np.abs(ref)
    assert ok.all()
    ok = np.abs(got_rows - rows) <= 1e-13 * rows
    assert ok.all()
    assert st["device_flags"] == 0
    assert st["events"] == (5 if rows.sum() > 0.0 else 0)
