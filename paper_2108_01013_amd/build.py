"""Build libdss.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libdss.so")
SOURCES = [os.path.join(CSRC, "dss_api.hip")]
HEADERS = [os.path.join(CSRC, h) for h in ("dss_kernels.hpp", "dss_adjoint.hpp", "dss_sized.hpp", "dss_lists.hpp", "dss_observe.hpp", "pair_vjp.hpp")] + [
    os.path.join(ROOT, "include", "dss.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-munsafe-fp-atomics",                                   # native global/LDS FP64 atomic add
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # no hoisting of instructions out of loops after selection: it moves the literal constants of
    # log and exp into registers for the whole loop, and the pair kernels spill (k_list, FP64, a
    # stress step at N = 100k 37.5 us with it, 27.9 without; at N = 500k 166 and 107)
    "-mllvm", "-disable-machine-licm",
    "-Wall", "-Wno-unused-function",
]


def build(verbose: bool = False) -> str:
    cmd = [HIPCC, *FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC, *SOURCES, "-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
