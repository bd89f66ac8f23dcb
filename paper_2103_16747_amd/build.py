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
    # and addresses hoisted out of it would hold registers in all phases, up to
    # the launch bound of 128 VGPRs (FP32) with 42 to 56 spilled and of 256 (FP64)
    # with up to 38 spilled, instead of 107 to 115 and 173 to 191 without a spill.
    # For the step kernels it is as good or better: the FP64 tile pass takes 122
    # VGPRs for 158 and 18.7 us for 19.8 (32 jobs on 20k tets), the FP32 one 120.5
    # us either way (256 jobs on 50k)
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
