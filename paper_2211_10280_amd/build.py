"""Builds libtensair.so (hand-written HIP for gfx950 + the C-ABI host code) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtensair.so")
SOURCES = ["api.hip", "sample.hip", "sort.hip", "grad.hip", "grad_sub.hip", "group.hip", "reduce.hip", "reduce_sub.hip", "apply.hip", "apply_ride.hip", "apply_chain.hip", "dense.hip", "probe.hip", "noalloc.hip"]
HEADERS = ["dev_common.h", "kernels.h", "aux_dev.h", "prep_dev.h", "apply_kernels.h", "rows_dev.h", "group_dev.h", "forward_dev.h", "reduce_dev.h", os.path.join("..", "..", "include", "tensair.h")]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off",                       # fused multiply-adds only where the source says fmaf
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(os.path.join(CSRC, f)) > t for f in SOURCES + HEADERS)


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every kernel and the host code into one shared library."""
    if not force and not stale():
        return LIB
    extra = os.environ.get("TENSAIR_EXTRA_HIPCC_FLAGS", "").split()   # tuning experiments (-DNAME=value)
    with tempfile.TemporaryDirectory() as tmp:      # one compiler per file, as many at a time as there are CPUs
        def compile_one(f):
            obj = os.path.join(tmp, f + ".o")
            cmd = ["hipcc", *FLAGS, *extra, "-c", os.path.join(CSRC, f), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.check_call(cmd)
            return obj

        with ThreadPoolExecutor(max(1, min(len(SOURCES), int(os.environ.get("MAX_JOBS", os.cpu_count() or 1))))) as pool:
            objs = list(pool.map(compile_one, SOURCES))
        subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
