"""Build the gfx950 HIP library ``libpsm.so`` in-tree with hipcc.

Usage: ``python -m paper_2303_11811_amd.build`` (or ``build()`` from Python).
Packed-FP32 instruction selection is disabled for all device code.
"""
from __future__ import annotations

import hashlib
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libpsm.so")
SOURCES = ["psm_kernels.hip", "psm_engine.cpp"]
ARCH = os.environ.get("PSM_OFFLOAD_ARCH", "gfx950")

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    f"-I{os.path.join(ROOT, 'include')}",
]


def source_hash() -> str:
    """Of the sources that decide how fast a launch is: the autotuner keeps its
    picks apart by it."""
    h = hashlib.sha256()
    for f in SOURCES + ["psm_internal.h"]:
        with open(os.path.join(CSRC, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:12]


def build(verbose: bool = False, extra_flags=None) -> str:
    """Compile every source and link libpsm.so (always rebuilds)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, src + ".o")
        cmd = [hipcc, *HIPCC_FLAGS, f'-DPSM_SOURCE_HASH="{source_hash()}"', *(extra_flags or []), "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        objs.append(obj)
    tmp = LIB + ".tmp"
    cmd = [hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv,
          extra_flags=["-Rpass-analysis=kernel-resource-usage"] if "--resources" in sys.argv else None)
