"""Transport in power-law disks whose exponents take roots and products (1/2,
1, 3/2) and in one that takes pow, against the oracle's step over the same
particles.  Bound 1e-12 as for the transport parity test: a few dozen FP64
roundings of a step whose kicks are the same random numbers; plus 1e-13 of the
starting height where the kick cancels it."""
import numpy as np
import pytest

import oracle as O
from paper_2507_21239_amd import workloads as W

from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p_exp,q_exp", [(1.0, 0.5), (1.5, 1.0), (0.5, 1.5), (0.7, 0.43)])
def test_transport_over_disk_exponents(p_exp, q_exp):
    from paper_2507_21239_amd import api
    say("disk exponents", p_exp, q_exp)
    work = W.c3_disk(seed=3, N=3000, n_r=10, n_z=10)
    prm, part = work["params"], work["particles"]
    prm.update(p=p_exp, q=q_exp, flags=[f for f in prm["flags"] if f != "coag"])
    rng = np.random.default_rng(4)
    part["m"][:] = 10.0 ** rng.uniform(-11.0, 3.0, len(part["m"]))
    dev = api.to_device(part)
    sim = api.Simulation(prm, dev, precision="fp64")
    sim.bin()
    dt = work["dt"] * 20
    sim.step(dt, 0, 1)
    got = {k: dev[k].cpu().numpy() for k in ("r", "z", "active")}
    sim.close()
    ref = {k: v.copy() if isinstance(v, np.ndarray) else v for k, v in part.items()}
    O.transport(prm, ref, 0, dt)
    assert np.array_equal(got["active"], ref["active"])
    for k in ("r", "z"):
        assert np.all(np.abs(got[k] - ref[k]) <= 1e-12 * np.abs(ref[k]) + 1e-13 * np.abs(part[k])), k
