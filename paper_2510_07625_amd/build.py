"""Builds libgato.so (the C-ABI library of include/gato.h) with hipcc for gfx950.

Each kernel translation unit is compiled separately (in parallel) and linked
into one shared library next to this file. Packed-FP32 instructions are kept
off (``-target-feature -packed-fp32-ops``).
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libgato.so")
ARCH = os.environ.get("GATO_OFFLOAD_ARCH", "gfx950")
SOURCES = ["sqp_mixed_f64.hip", "sqp_mixed_f32.hip", "sqp_long.hip", "sqp_n7.hip", "sqp_n6.hip", "sqp_n3.hip", "sqp_task.hip",
           "sqp_mixed_task.hip", "gato_api.hip", "gato_plant.hip", "gato_flops.cpp", "gato_probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]

# Loops on a 64-byte line, where it gains. The PCG loops are bound by instruction fetch
# from an unlucky start (8-byte instructions from 4 mod 8 bytes on): us per iteration,
# aligned against not: tip tracking 7 DoF N = 32 1.03 / 1.09; long solves 7 DoF N = 100
# on four workgroups 1.95 / 2.00, N = 128 on one 3.70 / 3.81; all-FP32 6 DoF N = 64
# 1.93 / 2.07. 7 DoF up to N = 64 1% slower and 3 DoF mixed (N = 32 all-FP32 5%
# slower, N = 128 4% faster): as they are.
ALIGNED = ("sqp_task.hip", "sqp_mixed_task.hip", "sqp_long.hip", "sqp_n6.hip")
EXTRA = {src: ["-falign-loops=64"] for src in ALIGNED}


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed on {src}")
    return obj


def build(jobs: int | None = None) -> str:
    os.makedirs(BUILD, exist_ok=True)
    jobs = jobs or min(len(SOURCES), max(1, (os.cpu_count() or 1)))
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    subprocess.run([HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp], check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
