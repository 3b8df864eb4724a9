"""Builds libsurf.so (the HIP library behind include/surf.h) in-tree for gfx950.

    python -m paper_2605_27534_amd.build

The kernel families with many instances are translation units of their own,
compiled once per precision (the 2D transport also once per number of rows a
wave takes); all units compile in parallel.
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libsurf.so")
PER_PRECISION = ["surf_batch_col2d.hip", "surf_col3d.hip", "surf_hj.hip"]
# (source, macros), the longest to compile first
UNITS = ([("surf_col2d.hip", ("SURF_REAL=" + r, "SURF_ROWS=%d" % n))
          for n in (8, 4, 2) for r in ("double", "float")]
         + [("surf_api.hip", ())]
         + [(f, ("SURF_REAL=" + r,)) for r in ("double", "float") for f in PER_PRECISION])

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # packed FP32 instructions stay off: ordinary float code only
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _compile(unit, out, verbose):
    src, macros = unit
    obj = os.path.join(out, "_".join([src[:-4], *(m.split("=")[1] for m in macros)]) + ".o")
    cmd = [HIPCC, *FLAGS, *("-D" + m for m in macros), "-c", "-o", obj, os.path.join(CSRC, src)]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return obj


def build(verbose: bool = False) -> str:
    tmp = LIB + ".tmp%d" % os.getpid()
    with tempfile.TemporaryDirectory() as out:
        with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
            objs = list(pool.map(lambda u: _compile(u, out, verbose), UNITS))
        cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp, *objs]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
    print(LIB)
