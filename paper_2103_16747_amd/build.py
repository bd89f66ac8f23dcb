"""Builds libfem.so (HIP, gfx950) in the package directory."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libfem.so")
SOURCES = [os.path.join(HERE, "csrc", "fem_lib.hip")]
DEPS = SOURCES + [os.path.join(HERE, "csrc", "fem_kernels.h"), os.path.join(HERE, "csrc", "layout.h"), os.path.join(HERE, "..", "include", "fem.h")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-munsafe-fp-atomics",
    # no packed-FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the persistent kernel inlines every solver phase into one loop: constants
    # and addresses hoisted out of it would hold registers in all phases
    # (FP32 154 VGPRs instead of 85, FP64 229 instead of 137)
    "-mllvm", "-disable-machine-licm",
    "-Wall", "-Wno-unused-result",
]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB_PATH + ".tmp"
    cmd = [hipcc, *HIPCC_FLAGS, "-o", tmp, *SOURCES]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True)
