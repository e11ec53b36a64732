"""Build the HIP shared library ``libfe_hip.so`` in-tree for gfx950.

Usage: ``python -m paper_1508_04596_amd.build`` (or ``build_library()``).
Every source under ``csrc/`` is compiled with hipcc for gfx950 only; packed
FP32 instructions are disabled for all device code.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libfe_hip.so")
SOURCES = ["fe_elem.hip", "fe_elem64.hip", "fe_vec.hip", "fe_mg.hip", "fe_filter.hip", "fe_mma.hip", "fe_noalloc.hip", "fe_batch.hip",
           "fe_api.cpp",
           "fe_solver.cpp", "fe_mg.cpp", "fe_topopt.cpp",
           "fe_serve.cpp", "fe_batch.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-x", "hip", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-I" + os.path.join(ROOT, "include"),
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-pragmas",
    # host code (coarse-grid band solves, Givens rotations): AVX2 + FMA, present
    # on every x86-64 host this library targets
    "-Xarch_host", "-mavx2", "-Xarch_host", "-mfma",
]


# The FP64 operator passes fill the 256 registers of two waves per SIMD; the
# scheduler's own pressure tracking keeps them within (registers spilled: J v 0
# instead of 10, J^T w 12 instead of 24).
FILE_FLAGS = {"fe_elem64.hip": ["-mllvm", "-amdgpu-use-amdgpu-trackers=1"]}


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, src + ".o")
    cmd = [HIPCC, *FLAGS, *FILE_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    return obj


def build_library(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(len(SOURCES), 8)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build_library(verbose=True)
    sys.exit(0)
