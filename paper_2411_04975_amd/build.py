"""Compile the HIP sources of the library for gfx950 into an in-tree shared object, and the Python
side's calls (csrc/sd_calls.cpp, host code) into another one beside it."""
from __future__ import annotations

import glob
import os
import subprocess

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB_PATH = os.path.join(_HERE, "libsd.so")
CALLS_PATH = os.path.join(_HERE, "_sdcalls.so")

# (Where several lanes add to one address the kernels let one lane do it.  The compiler's own code for that, around
# every atomic addition, stands in the way of a wave that is alone on its SIMD: decode steps of 64 requests 16.9 us with
# it and 16.6 without, drafts for 256 requests 17.5 and 17.2, for 512 20.3 and 19.8; for one no more than runs differ.)
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
    "-fno-fast-math", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None", "-Wno-unused-result",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(verbose: bool = False) -> str:
    """Always recompiles; returns the path of the shared object."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB_PATH + ".tmp.%d" % os.getpid()
    cmd = [hipcc] + HIPCC_FLAGS + ["-o", tmp] + sources()
    if verbose:
        print(" ".join(cmd))
    subprocess.check_call(cmd)
    os.replace(tmp, LIB_PATH)
    build_calls(verbose)
    return LIB_PATH


def build_calls(verbose: bool = False) -> str:
    import sysconfig
    import torch
    root = os.path.dirname(torch.__file__)
    tmp = CALLS_PATH + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wno-unused-result",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch.compiled_with_cxx11_abi()),
           "-I" + sysconfig.get_paths()["include"], "-I" + os.path.join(root, "include"),
           "-I" + os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-o", tmp, os.path.join(CSRC, "sd_calls.cpp"), "-L" + _HERE, "-l:libsd.so", "-Wl,-rpath,$ORIGIN",
           "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd))
    subprocess.check_call(cmd)
    os.replace(tmp, CALLS_PATH)
    return CALLS_PATH


if __name__ == "__main__":
    print(build(verbose=True))
