"""Compile the HIP sources into paper_2507_21239_amd/libmcd.so for gfx950.

hipcc cross-compiles without a GPU.  Flags: -O3, no FP contraction (the FP64
path keeps the operations of its formulas as they are written; FP32 code asks
for fused multiply-adds explicitly where it wants them), packed FP32
instructions disabled.  collide_ilp.hip and collide_ilp3.hip (the batched
kernels of the mixed form's common path) are also scheduled for
instruction-level parallelism; the other collision kernels and collide_ilp3.hip
sink instructions into the loops where they are used rather than spill their
results, but for collide_fp64_timed.hip and collide_generic_aux.hip, which run
faster without.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libmcd.so")
SOURCES = ["collide_batched.hip", "collide_batched_prob.hip", "collide_fp64.hip",
           "collide_fp64_timed.hip", "collide_generic_aux.hip", "collide_ilp.hip",
           "collide_ilp3.hip", "collide_plain.hip", "collide_plain_prob.hip", "capi.hip",
           "collide.hip", "binning.hip", "plan.hip", "transport.hip", "diagnostics.hip",
           "noalloc.hip"]
# per-file flags on top of CFLAGS
ILP = ["-mllvm", "--amdgpu-sched-strategy=max-ilp"]
SINK = ["-mllvm", "-sink-insts-to-avoid-spills=1"]
EXTRA = {"collide_fp64.hip": SINK, "collide_ilp.hip": ILP, "collide_ilp3.hip": ILP + SINK,
         "collide_batched.hip": SINK, "collide_batched_prob.hip": SINK, "collide_plain.hip": SINK,
         "collide_plain_prob.hip": SINK}
ARCH = os.environ.get("MCD_ARCH", "gfx950")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CFLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *CFLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    if verbose and r.stderr.strip():
        print(r.stderr, file=sys.stderr)
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
