"""Compile the HIP library libcxbwt.so in-tree for gfx950 with hipcc, and
libcxbwt_ceilings.so (the measurement kernel of bench.py --mode ceilings) and
libcxbwt_small.so (for tests: the library with the build by induced order taken
from far fewer bases on, so that the oracle can follow it)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = [os.path.join(HERE, "csrc", "cxbwt.hip")]
OUT = os.path.join(HERE, "libcxbwt.so")
CEILINGS_SOURCES = [os.path.join(HERE, "csrc", "ceilings.hip")]
CEILINGS_OUT = os.path.join(HERE, "libcxbwt_ceilings.so")
SMALL_OUT = os.path.join(HERE, "libcxbwt_small.so")
SMALL_FLAGS = ["-DCXBWT_INDUCE_MIN_BASES=60000ull", "-DCXBWT_INDUCE_TAIL_NS=1000000ull", "-DCXBWT_INDUCE_COLL_CHUNKS=20ull"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-Wall",
    # keep hipcc from forming packed-FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _hipcc(sources, out, verbose: bool, flags=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = out + ".tmp"
    cmd = [hipcc, *HIPCC_FLAGS, *flags, "-I", os.path.join(ROOT, "include"), *sources, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    errs = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{errs}")
    if verbose and errs.strip():
        print(errs, file=sys.stderr)
    os.replace(tmp, out)
    return out


def build(verbose: bool = False) -> str:
    with ThreadPoolExecutor(3) as pool:
        jobs = [pool.submit(_hipcc, CEILINGS_SOURCES, CEILINGS_OUT, verbose), pool.submit(_hipcc, SOURCES, OUT, verbose),
                pool.submit(_hipcc, SOURCES, SMALL_OUT, verbose, SMALL_FLAGS)]
        for j in jobs:
            j.result()
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
