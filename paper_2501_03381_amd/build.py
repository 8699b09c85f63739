"""Build libthoi.so (HIP for gfx950) in-tree with hipcc.

Every HIP translation unit is compiled for gfx950 only, with packed FP32 instructions
disabled (``-Xclang -target-feature -Xclang -packed-fp32-ops``), and linked into one shared
library next to this file.  ``python -m paper_2501_03381_amd.build`` rebuilds it.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libthoi.so")
SOURCES = ["nplets_bwd_lane_hi.hip", "nplets_bwd_lane_lo.hip", "nplets_fwd.hip", "nplets_prefix.hip", "nplets_cube.hip", "nplets_cube_verify.hip", "nplets_cube_gate.hip", "nplets_wave2.hip", "nplets_multi.hip",
           "api.cpp", "fan.cpp",
           "copula.hip", "cov.hip", "nplets_bwd.hip",
           "objective.hip", "reduce_final.hip", "noalloc.hip", "nplets_anneal.hip", "nplets_greedy.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-I", CSRC, "-I", INCLUDE,
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
