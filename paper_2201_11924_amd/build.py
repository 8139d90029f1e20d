"""Builds the gfx950 shared library ``libsimsense.so`` in-tree with hipcc.

Every HIP source under ``csrc/`` is compiled to an object (in parallel), then
linked into one shared object next to this file.  No torch, no JIT cache.
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsimsense.so")
ARCH = "gfx950"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-ffp-contract=off",
    # keep the compiler from forming packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
    "-Wno-unused-command-line-argument",
]


# Per-file additions.  The fused net inference keeps its MFMA accumulators in
# the vector registers its epilogues read (the default places them in the
# accumulation registers and copies every result across).
# The aggregation's steps are serial chains with DPP moves, which need idle issue
# slots after the instruction that makes their source: the ILP scheduler fills them
# with other steps' independent work (the default one, after low register counts,
# leaves 3 times the s_nops).  Loops start on a cache line: where a kernel's loops fall
# otherwise moves with every instruction before them (one s_nop at the kernel's start:
# 320x240, D = 64 53.2 -> 52.4 us a call, 500x375, D = 48 99.8 -> 101.6; three: 960x540,
# D = 96 171 -> 175; aligned 52.9, 100.0, 171).
_ILP = ["-mllvm", "-amdgpu-sched-strategy=max-ilp", "-falign-loops=64"]
FILE_FLAGS = {
    "net_infer.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "sgbm.hip": _ILP,
    **{f"agg_dpl{n}.hip": _ILP for n in (1, 2, 4, 6, 8, 12, 16)},
}


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.basename(src) + ".o")
    cmd = [HIPCC, *FLAGS, *FILE_FLAGS.get(os.path.basename(src), []), "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    srcs = sources()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs,
           "-L/opt/rocm/lib", "-lrocprofiler-sdk-roctx", "-Wl,-rpath,/opt/rocm/lib"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
