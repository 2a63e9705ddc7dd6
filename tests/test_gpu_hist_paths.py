"""Both paths of the sigma_d(m, r) histogram -- bins in LDS, in one part or
several, and atomics on global memory -- against the oracle at the edges of
their dispatch: counts bit-exact, masses within the reordering bound of FP64
sums (relative 2 * count * 2^-53 per bin)."""
import numpy as np
import pytest

import oracle as O
from paper_2507_21239_amd import workloads as W

from gpu_common import say

pytestmark = pytest.mark.gpu

AU = W.AU


@pytest.mark.parametrize("N,n_rb,n_mb,linear", [
    (64_000, 128, 100, False),    # the largest histogram in one part, on the line of N = 5 bins
    (63_999, 128, 100, False),    # below it: atomics
    (65_537, 129, 100, False),    # one radial row in a second part, a ragged last round
    (240_000, 511, 90, False),    # four parts
    (300_000, 569, 90, False),    # five: atomics
    (100_000, 8, 900, True),      # edges in no geometric progression: the guess misses
    (150_000, 1010, 12, False),   # 1024 edges
    (150_000, 1011, 12, False),   # 1025 edges: atomics
    (150_000, 1, 1000, False),    # a single radial row
    (100_000, 4, 6400, False),    # two rows a part would fit, the edges do not: atomics
    (2049, 2, 2, False),          # three workgroups
    (1, 1, 1, False),
])
def test_histogram_paths_match_oracle(N, n_rb, n_mb, linear):
    from paper_2507_21239_amd import api
    say("histogram paths", N, n_rb, n_mb, linear)
    rng = np.random.default_rng(N + n_rb)
    part = W._particles(N)
    part["r"][:] = AU * 10.0 ** rng.uniform(-0.2, 2.2, N)
    part["m"][:] = 10.0 ** rng.uniform(-12.5, 3.0, N)
    part["M"][:] = rng.uniform(0.1, 3.0, N) * 1e21
    part["active"][:] = (rng.random(N) > 0.07).astype(np.uint8)
    space = np.linspace if linear else np.geomspace
    re = AU * space(0.0 if linear else 1.0, 100.0, n_rb + 1)
    me = space(1e-12, 1e2, n_mb + 1)
    k = min(N, 64)  # on edges, and just below them
    part["r"][:k] = re[np.linspace(0, n_rb, k).astype(int)]
    part["m"][:k] = me[np.linspace(0, n_mb, k).astype(int)]
    part["r"][1:k:2] = np.nextafter(part["r"][1:k:2], 0.0)
    sim = api.Simulation(W.benchmark_params(), api.to_device(part), precision="mixed")
    sig, cnt = sim.sigma_hist(re, me)
    again, _ = sim.sigma_hist(re, me)
    sig, cnt = sig.cpu().numpy(), cnt.cpu().numpy().view(np.uint32)
    again = again.cpu().numpy()
    sim.close()
    osig, ocnt, n = O.sigma_hist(part, re, me)
    assert (n > 0 or N == 1) and np.array_equal(cnt, ocnt)
    bound = 2.0 * np.maximum(ocnt, 1) * 2.0 ** -53 * np.abs(osig)
    for got in (sig, again):
        assert np.all(np.abs(got - osig) <= bound + 1e-300)
