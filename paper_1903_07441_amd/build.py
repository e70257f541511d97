"""Build libtwg.so for gfx950 with hipcc (in-tree, no JIT cache).

    python -m paper_1903_07441_amd.build
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libtwg.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

# Packed FP32 ops are disabled on purpose; contraction is off so that every
# rounding in the kernels is the one written in the source (explicit fmaf
# calls are kept).
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # a kernel's first arguments arrive in registers (k_relax_slot's control
    # block and slot number)
    "-mllvm", "-amdgpu-kernarg-preload-count=3",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# sources whose kernels are instantiated per sweep depth: compiled once
# without TWG_DEPTH (everything else) and once for each depth
DEPTH_SOURCES = ("solve.hip", "sor_stream.hip", "batch.hip")
DEPTHS = range(1, 9)


def _compile(job) -> str:
    src, depth = job
    obj = os.path.join(OBJ, os.path.basename(src) + (f".d{depth}" if depth else "") + ".o")
    cmd = [HIPCC, *FLAGS, *([f"-DTWG_DEPTH={depth}"] if depth else []), "-c", src, "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{res.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    jobs = [(s, 0) for s in srcs]
    # the deepest kernels take longest: first in the queue
    jobs = [(s, d) for d in reversed(DEPTHS) for s in srcs if os.path.basename(s) in DEPTH_SOURCES] + jobs
    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(_compile, jobs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
