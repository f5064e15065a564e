"""Builds liboasmc.so (the HIP library behind include/oasmc.h) in-tree for gfx950."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "liboasmc.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    # packed fp32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-Wall", "-Wno-unused-result",
]

# The step kernels' loops over tiles and steps hold the constants of every
# polynomial in them (exp, log, sin): hoisted out of the loops they take some 45
# registers a lane for the whole kernel, and what spills for them costs more than
# the moves saved (a logistic-regression run 664 -> 648 ms, the d = 100 mixture
# HMC step 155 -> 126 us, a d = 100 Gaussian MALA run 6.0 -> 4.4 ms).  The
# other sources hold no such loop.  The option is LLVM's own: a compiler without it
# stops the build, and the waves per SIMD of the step kernels (MinWaves, SweepWaves)
# were chosen with it, so they are to be measured again if it goes.
IN_PLACE_CONSTANTS = ["-mllvm", "-disable-machine-licm"]
IN_PLACE_SOURCES = ("valu_", "sweep_logreg", "adjoint")


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    in_place = os.path.basename(src).startswith(IN_PLACE_SOURCES)
    cmd = [HIPCC, *FLAGS, *(IN_PLACE_CONSTANTS if in_place else []), "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed on {src}")
    return obj


def build(jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))
    with ThreadPoolExecutor(max_workers=min(jobs, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("link failed")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
