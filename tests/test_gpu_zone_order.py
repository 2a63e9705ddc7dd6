"""Order of the particles inside a zone, (z, index), from the zone sort's
32-bit network, its runs of equal reduced heights and the 64-bit network that
takes over where those are long, against the oracle: exact."""
import numpy as np
import pytest

import oracle as O
from paper_2507_21239_amd import workloads as W

from gpu_common import say

pytestmark = pytest.mark.gpu

AU = W.AU


def _heights(kind, N, rng):
    z = AU * 10.0 ** rng.uniform(-9, 0, N)
    if kind == "equal":
        z[:] = 0.3 * AU
    elif kind == "ulps":        # no bits to drop: all within a few thousand ulps
        z = AU + rng.integers(0, 3000, N) * np.spacing(AU)
    elif kind == "clusters":    # two heights far apart, ulps inside each
        z = np.where(rng.random(N) < 0.5, 1e-9 * AU, AU) * (1.0 + rng.integers(0, 500, N) * 2.0 ** -52)
    elif kind == "runs":        # runs of 2 .. 17 equal or nearly equal heights
        k = np.arange(N) // 17
        z = z[k] * (1.0 + rng.integers(0, 3, N) * 2.0 ** -51)
    return z


@pytest.mark.parametrize("kind", ["spread", "equal", "ulps", "clusters", "runs"])
@pytest.mark.parametrize("N,n_r", [(4, 1), (9, 1), (511, 1), (512, 1), (513, 1), (2048, 1), (3 * 700, 3),
                                   (4097, 1), (8192, 1), (100_003, 50)])
def test_zone_order_is_exact(kind, N, n_r):
    from paper_2507_21239_amd import api
    say("zone order", kind, N, n_r)
    rng = np.random.default_rng(N)
    p = W.benchmark_params(n_r=n_r, n_z=4)
    r = AU * 10.0 ** rng.uniform(0, 2, N)
    z = _heights(kind, N, rng)
    active = np.ones(N, dtype=np.uint8)
    part = dict(r=r, z=z, m=np.full(N, 1e-11), M=np.ones(N), active=active)
    sim = api.Simulation(p, api.to_device(part), precision="mixed")
    sim.bin()
    order = sim.cells()["order"].cpu().numpy()
    sim.close()
    assert np.array_equal(order, O.bin_particles(p, r, z, active)["order"])
