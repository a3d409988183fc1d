"""Build libgbp.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2308_08410_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgbp.so")
SOURCES = ["plan.cpp", "profile.cpp", "eikonal.hip", "walk.hip", "ecg.hip", "optim.hip", "step.cpp", "mlp.hip", "points.hip", "local.hip", "leadfield.hip", "tri.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
    # keep the compiler from emitting packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the network's initialisation draws 201,000 normals on the host: 9 ms, 15 where the
    # linker happens to put the generator across a 32-byte boundary
    "-Xarch_host", "-falign-functions=32",
    "-Wno-unused-result", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


def build(verbose: bool = False) -> str:
    srcs = []
    for s in SOURCES:
        p = os.path.join(CSRC, s)
        if s.endswith(".cpp"):
            srcs += ["-x", "hip", p]
        else:
            srcs += ["-x", "hip", p]
    tmp = LIB + ".tmp"
    cmd = [HIPCC] + FLAGS + srcs + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    print(LIB)
