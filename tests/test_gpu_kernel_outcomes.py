"""The test kernels know no velocities and no fragmentation: every event of
theirs sticks, in both precisions and schedules, also where the fragmentation
velocity is too small for FP32."""
import numpy as np
import pytest

from paper_2507_21239_amd import workloads as W

from gpu_common import run_gpu_explicit

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kernel", ["constant", "linear"])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("schedule", ["plain", "batched"])
def test_test_kernels_only_stick(kernel, precision, schedule):
    work = W.c1_single_cell(seed=2, n=100, t_end=50.0)
    work["params"].update(kernel=kernel, v_frag=1e-60)
    work.update(dt=0.0, max_events=80)
    start = work["particles"]["m"].copy()
    part, st, _ = run_gpu_explicit(work, precision, schedule)
    assert st["events"] == 80 and st["outcomes"] == [80, 0, 0, 0]
    assert np.all(part["m"] >= start) and part["m"].sum() > start.sum()
