"""Builds the HIP library ``libgl_hip.so`` (gfx950) in-tree.

    python -m paper_2410_05408_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libgl_hip.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = os.environ.get("GL_OFFLOAD_ARCH", "gfx950")

FLAGS = [
    "-O3", "-std=c++17", f"--offload-arch={ARCH}", "-fPIC", "-shared",
    # packed FP32 instructions are kept out of every code object
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # literals and set constants hoisted out of the fused pass's loops by machine
    # LICM spill (74 registers per lane against 28 without it)
    "-mllvm", "-disable-machine-licm",
    "-Wall", "-Wno-unused-function",
]


def build(verbose: bool = False, out: str = LIB, defines=()) -> str:
    """Compiles the library to ``out``; ``defines`` are extra -D macros
    (e.g. GL_ARC_TOL=1e-7)."""
    srcs = [os.path.join(CSRC, "gl_lib.hip"), os.path.join(CSRC, "gl_mlp.hip"),
            os.path.join(CSRC, "gl_mcmc.hip"), os.path.join(CSRC, "gl_io.cpp")]
    cmd = [HIPCC, *FLAGS, *[f"-D{d}" for d in defines], "-I", os.path.join(ROOT, "include"),
           "-I", CSRC, *srcs, "-o", out + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(out + ".tmp", out)
    return out


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
