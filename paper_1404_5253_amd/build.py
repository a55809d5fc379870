"""Build libwpcd.so (host C++ + gfx950 HIP kernels) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libwpcd.so")
SOURCES = ["host_math.cpp", "capi.cpp", "mixed.cpp", "batch.cpp", "observables.cpp", "kernels.hip", "kernels_mixed.hip",
           "spmm_f32.hip", "spmm_f64.hip", "spmm_f32v_f64x.hip", "noalloc.hip"]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc"):
        if c and os.path.exists(c):
            return c
    return "hipcc"


def _jobs() -> int:
    """Compilers at a time: MAX_JOBS where it is a positive number, else 8."""
    n = os.environ.get("MAX_JOBS", "").strip()
    return int(n) if n.isdigit() and int(n) > 0 else 8


def _run(cmds, over, verbose):
    if verbose:
        for c in cmds:
            print(" ".join(c), flush=True)
    for r in list(over(lambda c: subprocess.run(c, capture_output=True, text=True), cmds)):
        if r.returncode != 0:
            sys.stderr.write(r.stdout + r.stderr)
            raise RuntimeError("hipcc failed building libwpcd.so")


def build(verbose: bool = False) -> str:
    """Compile every source into paper_1404_5253_amd/libwpcd.so (always recompiles)."""
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    cc = [hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
          # packed FP32 instructions are kept out of every kernel
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument"]
    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as work:
        objs = [os.path.join(work, os.path.basename(s) + ".o") for s in srcs]
        cmds = [cc + ["-c", s, "-o", o] for s, o in zip(srcs, objs)]
        with ThreadPoolExecutor(_jobs()) as pool:
            _run(cmds, pool.map, verbose)
        _run([cc + ["-shared", "-o", tmp] + objs + ["-lpthread"]], map, verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
