"""Accuracy of the powers x^-e of the power-law disk that transport forms from
roots and products, compiled here for the host from the kernels' own source and
compared with 64-bit-mantissa long doubles: half an ulp for the last rounding,
and 0.005 ulp for the long doubles' own."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCE = """
#include "physics.hpp"
extern "C" void powers(const double *x, double e, double *y, long n) {
  for (long k = 0; k < n; ++k) y[k] = mcd::inverse_power(x[k], e);
}
"""


@pytest.fixture(scope="module")
def powers(tmp_path_factory):
    if shutil.which(HIPCC) is None:
        pytest.skip("no hipcc")
    if np.finfo(np.longdouble).nmant < 63:
        pytest.skip("no long double beyond double")
    d = tmp_path_factory.mktemp("powers")
    src, so = str(d / "powers.hip"), str(d / "powers.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([HIPCC, "--cuda-host-only", "-O2", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2507_21239_amd", "csrc"), src, "-o", so], check=True)
    f = ctypes.CDLL(so).powers
    f.argtypes = [ctypes.c_void_p, ctypes.c_double, ctypes.c_void_p, ctypes.c_long]

    def call(x, e):
        x = np.ascontiguousarray(x, dtype=np.float64)
        y = np.empty_like(x)
        f(x.ctypes.data, e, y.ctypes.data, len(x))
        return y
    return call


@pytest.mark.parametrize("e", [0.5, 1.0, 1.5])
@pytest.mark.parametrize("lo,hi", [(1.0, 100.0), (0.9, 1.1), (1e-80, 1e80)])
def test_half_integer_powers_are_correct_to_the_last_rounding(powers, e, lo, hi):
    x = np.exp(np.random.default_rng(5).uniform(np.log(lo), np.log(hi), 200_000))
    y = powers(x, e)
    X = x.astype(np.longdouble)
    ref = 1 / {0.5: np.sqrt(X), 1.0: X, 1.5: X * np.sqrt(X)}[e]
    ulps = np.abs(y.astype(np.longdouble) - ref) / np.spacing(ref.astype(np.float64))
    assert ulps.max() <= 0.505, float(ulps.max())


@pytest.mark.parametrize("e", [0.5, 1.0, 1.5, 0.43])
def test_powers_outside_any_disk(powers, e):
    x = np.array([0.0, 1e-300, 1e-95, 1e95, 1e300, np.inf, np.nan, -1.0])
    with np.errstate(all="ignore"):
        assert np.allclose(powers(x, e), np.power(x, -e), rtol=1e-14, atol=0.0, equal_nan=True)
