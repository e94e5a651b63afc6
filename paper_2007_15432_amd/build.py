"""Build libp3t.so (all HIP kernels + the C ABI) for gfx950 with hipcc.

Objects go to paper_2007_15432_amd/_build/, the library to
paper_2007_15432_amd/libp3t.so.  Packed FP32 instructions are disabled at
code generation (-packed-fp32-ops).
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libp3t.so")
ARCH = os.environ.get("P3T_OFFLOAD_ARCH", "gfx950")

SOURCES = ["util.hip", "cutoff.hip", "tree.hip", "walk.hip", "force.hip", "force_split.hip", "nbr.hip", "hermite.hip",
           "adjoint.hip", "slow.hip", "kepler.hip", "energy.hip", "merge.hip", "api.hip"]

CFLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(HERE, "..", "include"),
]
# hermite.hip: instruction order chosen for independent work between dependent
# FP64 operations rather than for occupancy (its long chains run on one
# wavefront per SIMD); the instructions and their results are the same.  The
# force kernels run three or four wavefronts per SIMD and are no faster with it
# (200,000 particles 490 us an evaluation, 484 without; 2^20 1685 and 1675, mixed
# 1363 and 1360).
FILE_FLAGS = {"hermite.hip": ["-mllvm", "-amdgpu-sched-strategy=max-ilp"]}


def hipcc() -> str:
    p = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(p):
        raise RuntimeError("hipcc not found")
    return p


def _compile(src: str) -> str:
    obj = os.path.join(OUT, os.path.splitext(src)[0] + ".o")
    cmd = [hipcc(), *CFLAGS, *FILE_FLAGS.get(src, []), "-c", os.path.join(SRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr[-6000:]}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(OUT, exist_ok=True)
    srcs = [s for s in SOURCES if os.path.exists(os.path.join(SRC, s))]
    jobs = min(len(srcs), max(1, min(8, os.cpu_count() or 1)))
    with cf.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr[-4000:]}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
