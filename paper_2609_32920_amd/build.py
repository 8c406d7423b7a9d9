"""Compile the HIP library liblt.so for gfx950 (in-tree, next to this file)."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblt.so")
LIB_COUNTERS = os.path.join(HERE, "liblt_counters.so")
SOURCES = ["lt_attached.hip", "lt_kernels.hip", "lt_guide.hip", "lt_api.cpp"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # no packed-FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable", "-Wno-unused-value",
]


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)


def build(verbose: bool = False) -> str:
    """Product library plus the diagnostic counters build; the sources of both
    are compiled side by side."""
    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(max_workers=8) as pool:
        jobs, objs = [], {}
        for out, extra in ((LIB, []), (LIB_COUNTERS, ["-DLT_COUNTERS"])):
            for src in SOURCES:
                obj = os.path.join(tmp, f"{os.path.basename(out)}.{src}.o")
                objs.setdefault(out, []).append(obj)
                # .cpp files are host+device HIP sources as well
                jobs.append(pool.submit(_run, [HIPCC, "-x", "hip", *FLAGS, *extra, "-I", os.path.join(ROOT, "include"),
                                               "-I", CSRC, "-c", os.path.join(CSRC, src), "-o", obj], verbose))
        for j in jobs:
            j.result()
        for out, o in objs.items():
            _run([HIPCC, "--offload-arch=gfx950", "-shared", "-o", out + ".tmp", *o], verbose)
            os.replace(out + ".tmp", out)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
