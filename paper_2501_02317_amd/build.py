"""Compile the HIP library libhydro.so for gfx950 (in-tree).

    python -m paper_2501_02317_amd.build

Flags: gfx950 only; no implicit FP contraction (the kernels place their
fused multiply-adds and Newton-refined reciprocals by hand, so the FP64 path
agrees with the oracle to rounding); packed FP32 instructions disabled.
"""
import concurrent.futures
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libhydro.so")
# (source, part): kernels.hip compiles in parts (its HYDRO_PART), so the parts
# compile side by side
UNITS = [("csrc/kernels.hip", p) for p in (6, 5, 4, 3, 2, 1, 0)] + [("csrc/runtime.hip", 0), ("csrc/plan.cpp", 0)]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-parameter",
]


def build(force=True, extra=(), verbose=False):
    """Compile libhydro.so; with force=False only when it is missing."""
    if not force and os.path.exists(LIB):
        return LIB
    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as d:
        def compile_unit(unit):
            src, part = unit
            obj = os.path.join(d, f"{os.path.basename(src)}.{part}.o")
            cmd = [HIPCC, *FLAGS, *extra, f"-DHYDRO_PART={part}", "-I", os.path.join(ROOT, "include"),
                   "-I", os.path.join(HERE, "csrc"), "-c", os.path.join(HERE, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj

        with concurrent.futures.ThreadPoolExecutor(min(8, len(os.sched_getaffinity(0)))) as pool:
            objs = list(pool.map(compile_unit, UNITS))
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(force=True, extra=sys.argv[1:], verbose=True))
