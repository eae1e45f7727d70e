"""Build libbload.so (the C-ABI HIP library), libbload_yardsticks.so (plain streaming
kernels that a benchmark times beside it) and libbload_scan_nowait.so (the scan with a bound of 0
on its wait, for a test) in-tree for gfx950.

    python -m paper_2310_10879_amd.build

hipcc cross-compiles without a GPU present.  The shared objects land next to
this file so that the bindings, and a copy of the tree on another machine, find
them without any install step.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libbload.so")
YS_SRC = os.path.join(PKG, "yardsticks", "bload_yardsticks.hip")
YS_LIB = os.path.join(PKG, "libbload_yardsticks.so")
NOWAIT_LIB = os.path.join(PKG, "libbload_scan_nowait.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
    # keep the compiler from fusing float pairs into packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]
# Flags of single sources.  The chain of draws is one wavefront in one loop, and where that lies across a border of
# instruction fetches it is 2 to 4 % slower.
OWN_FLAGS = {"bload_random_fit.hip": ["-falign-loops=64"]}


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(verbose: bool = True) -> str:
    """Every source file to an object, side by side, then the libraries from them."""
    with tempfile.TemporaryDirectory() as tmp:
        def compile_one(job):
            src, out, extra = job
            cmd = [HIPCC] + FLAGS + extra + ["-c", "-o", os.path.join(tmp, out), src]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.check_call(cmd)
            return os.path.join(tmp, out)

        api, scan = os.path.join(CSRC, "bload_api.hip"), os.path.join(CSRC, "bload_scan.hip")
        jobs = [(scan, "nowait.o", ["-DBLOAD_SCAN_POLLS=0"])] + \
            [(src, os.path.basename(src) + ".o", OWN_FLAGS.get(os.path.basename(src), [])) for src in sources()] + [(YS_SRC, "yardsticks.o", [])]
        jobs.sort(key=lambda job: -os.path.getsize(job[0]))          # the longest first
        with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
            objects = dict(zip((job[1] for job in jobs), pool.map(compile_one, jobs)))
        for lib, parts in ((LIB, [os.path.basename(src) + ".o" for src in sources()]), (YS_LIB, ["yardsticks.o"]),
                           (NOWAIT_LIB, ["nowait.o", os.path.basename(api) + ".o"])):
            cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib] + [objects[part] for part in parts]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    build()
    print("built", LIB, "and", YS_LIB)
    sys.exit(0)
