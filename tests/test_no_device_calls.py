"""The built kernels call no functions: a pair of particles evaluated by a call
passes its records through memory (one such kernel ran its row sums seven times
slower than its neighbours).  Every function symbol of the library's gfx950 code
is a kernel, with its descriptor beside it."""
import glob
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2507_21239_amd", "libmcd.so")
BIN = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


def test_every_function_of_the_device_code_is_a_kernel(tmp_path):
    tools = [os.path.join(BIN, t) for t in ("llvm-objdump", "llvm-readelf")]
    if not os.path.exists(LIB) or not all(shutil.which(t) for t in tools):
        pytest.skip("needs the built library and the ROCm binutils")
    lib = shutil.copy(LIB, tmp_path)
    subprocess.run([tools[0], "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    objs = glob.glob(str(tmp_path / "*gfx950"))
    assert objs
    kernels, others = 0, []
    for o in objs:
        out = subprocess.run([tools[1], "-sW", o], check=True, capture_output=True, text=True).stdout
        rows = [line.split() for line in out.splitlines()]
        names = {r[7] for r in rows if len(r) > 7}
        funcs = {r[7] for r in rows if len(r) > 7 and r[3] == "FUNC"}
        kernels += len(funcs)
        others += sorted(f for f in funcs if f + ".kd" not in names)
    assert kernels > 40 and others == []
