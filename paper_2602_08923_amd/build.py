"""Compile libdq.so (the HIP kernels + C ABI) for gfx950, in-tree.

hipcc cross-compiles without a GPU.  Flags that matter for bit-exactness against the CPU
oracle: -ffp-contract=off (fused multiply-adds only where the source writes them) and the
default correctly rounded fp32 division; packed-fp32 instructions are disabled, and so is the fold of
shifts and masks into SDWA operands (an SDWA instruction takes the issue slots of three simple ones here).
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdq.so")
SOURCES = ["dq_kernels.hip", "dq_walk.hip", "mx_kernels.hip", "pp_kernels.hip", "probe_kernels.hip", "dq_api.cpp", "dq_replay.cpp"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-sdwa-peephole=0",
    "-Wall", "-Wno-unused-function",
]


def build(verbose=False, extra_flags=()):
    srcs = [os.path.join(CSRC, s) for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    cmd = ["hipcc", "-x", "hip"] + FLAGS + list(extra_flags) + ["-I", os.path.join(ROOT, "include"), "-I", CSRC] + srcs + ["-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, extra_flags=sys.argv[1:]))
