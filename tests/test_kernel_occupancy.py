"""Registers of the built collision kernels.  A CU's SIMD holds 512 of them a
lane: the mixed form's batched kernels stay within the 168 of three waves, but for
the time-limited ones without the composition mix (256, two waves), as do all of
the FP64 form.  With two waves instead of three, 2500 cells of the test kernel take
1.4 times as long."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2507_21239_amd", "libmcd.so")
BIN = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
# collide_batched<rate type, slots a lane, fast, probabilistic, fractions or log, event budget>
NAME = re.compile(r"collide_batchedI([fd])Li(\d)ELb([01])ELb([01])ELb([01])ELi([012])E")


def test_batched_kernels_keep_their_waves(tmp_path):
    tools = [os.path.join(BIN, t) for t in ("llvm-objdump", "llvm-readelf")]
    if not os.path.exists(LIB) or not all(shutil.which(t) for t in tools):
        pytest.skip("needs the built library and the ROCm binutils")
    lib = shutil.copy(LIB, tmp_path)
    subprocess.run([tools[0], "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    seen = {}
    for o in glob.glob(str(tmp_path / "*gfx950")):
        out = subprocess.run([tools[1], "--notes", o], check=True, capture_output=True, text=True).stdout
        name = None
        for line in out.splitlines():
            key, _, val = line.strip().lstrip("- ").partition(":")
            if key == ".name" and NAME.search(val):
                name = val.strip()
            elif key == ".vgpr_count" and name:
                seen[name] = int(val)
                name = None
            elif key == ".symbol":
                name = name if name and val.strip().startswith(name) else None
    assert len(seen) >= 24
    for name, vgpr in seen.items():
        rt, _, _, _, aux, limit = NAME.search(name).groups()
        two = rt == "d" or (aux == "0" and limit == "1")
        assert vgpr <= (256 if two else 168), (name, vgpr)
