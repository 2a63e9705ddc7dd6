"""Histograms of up to 4096 bins, which are in LDS for any number of particles
and edges, against the oracle at the edges of that rule: from fewer particles
than a row of scratch holds bins (one workgroup, which writes the outputs) to
thousands of edges on one axis, and with all particles in one bin.  Counts
bit-exact, masses within the reordering bound of FP64 sums."""
import numpy as np
import pytest

import oracle as O
from paper_2507_21239_amd import workloads as W

from gpu_common import say

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

AU = W.AU


@pytest.mark.parametrize("where", ["spread", "one"])
@pytest.mark.parametrize("N,n_rb,n_mb", [
    (1, 64, 64), (50, 64, 64),      # one workgroup
    (3071, 64, 64), (3072, 64, 64), (3073, 64, 64),   # about a row of scratch
    (20_479, 64, 64),               # below 5 particles a bin
    (20_484, 17, 241),              # 4097 bins: below it, atomics
    (50_000, 4096, 1), (50_000, 1, 4096), (50_000, 1365, 3),   # thousands of edges
    (500, 4096, 1),
])
def test_few_bins_match_the_oracle(N, n_rb, n_mb, where):
    from paper_2507_21239_amd import api
    say("few bins", N, n_rb, n_mb, where)
    rng = np.random.default_rng(N + n_rb)
    part = W._particles(N)
    part["r"][:] = AU * 10.0 ** rng.uniform(-0.1, 2.1, N) if where == "spread" else 7.0 * AU
    part["m"][:] = 10.0 ** rng.uniform(-12.5, 2.5, N) if where == "spread" else 1e-7
    part["M"][:] = rng.uniform(0.1, 3.0, N) * 1e21
    part["active"][:] = (rng.random(N) > 0.07).astype(np.uint8)
    re, me = AU * np.geomspace(1.0, 100.0, n_rb + 1), np.geomspace(1e-12, 1e2, n_mb + 1)
    sim = api.Simulation(W.benchmark_params(), api.to_device(part), precision="mixed")
    sig, cnt = sim.sigma_hist(re, me)
    sig, cnt = sig.cpu().numpy(), cnt.cpu().numpy().view(np.uint32)
    bare = torch.full((n_rb, n_mb), np.nan, dtype=torch.float64, device="cuda")   # no counts wanted
    sim._check(sim.lib.mcd_sigma_hist(sim.ctx, re.ctypes.data, n_rb, me.ctypes.data, n_mb,
                                      bare.data_ptr(), None), "mcd_sigma_hist")
    bare = bare.cpu().numpy()
    sim.close()
    osig, ocnt, _ = O.sigma_hist(part, re, me)
    assert np.array_equal(cnt, ocnt)
    # FP64 sums of positive terms in any order, then one division
    bound = 2.0 * np.maximum(ocnt, 1) * 2.0 ** -53 * np.abs(osig)
    for got in (sig, bare):
        ok = np.abs(got - osig) <= bound
        assert ok.all()
