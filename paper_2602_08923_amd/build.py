"""Compile libdq.so (the HIP kernels + C ABI) for gfx950 and _dqpy.so (the binding's native half), in-tree.

hipcc cross-compiles without a GPU.  Flags that matter for bit-exactness against the CPU
oracle: -ffp-contract=off (fused multiply-adds only where the source writes them) and the
default correctly rounded fp32 division; packed-fp32 instructions are disabled, and so is the fold of
shifts and masks into SDWA operands (an SDWA instruction takes the issue slots of three simple ones here).
"""
import os
import subprocess
import sys
import sysconfig
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdq.so")
EXT = os.path.join(HERE, "_dqpy.so")
SOURCES = ["dq_kernels.hip", "dq_few.hip", "dq_walk.hip", "dq_thin.hip", "dq_bounds.hip", "mx_kernels.hip", "pp_kernels.hip", "probe_kernels.hip", "dq_api.cpp", "dq_replay.cpp"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-sdwa-peephole=0",
    "-Wall", "-Wno-unused-function",
]


def _run(cmds, verbose):
    """Run the commands side by side; raise if one fails."""
    procs = []
    for cmd in cmds:
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((cmd, subprocess.Popen(cmd)))
    for cmd, p in procs:
        if p.wait() != 0:
            for _, other in procs:
                other.wait()
            raise subprocess.CalledProcessError(p.returncode, cmd)


def _extension_command():
    """The host compiler's command for _dqpy.so, against this interpreter's and PyTorch's headers."""
    import torch
    t = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
            "-I", sysconfig.get_path("include"), "-isystem", os.path.join(t, "include"),
            "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"), "-isystem", os.path.join(rocm, "include"),
            "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, "dq_python.cpp"), "-o", EXT,
            "-L", os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]


def build(verbose=False, extra_flags=()):
    with tempfile.TemporaryDirectory() as tmp:
        cmds, objs = [_extension_command()], []
        for s in SOURCES:
            objs.append(os.path.join(tmp, s + ".o"))
            cmds.append(["hipcc", "-x", "hip"] + [f for f in FLAGS if f != "-shared"] + list(extra_flags) +
                        ["-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", os.path.join(CSRC, s), "-o", objs[-1]])
        _run(cmds, verbose)
        _run([["hipcc", "--offload-arch=gfx950", "-fPIC", "-shared"] + objs + ["-o", LIB]], verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, extra_flags=sys.argv[1:]))
