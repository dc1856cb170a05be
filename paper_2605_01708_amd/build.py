"""Builds, in-tree, libsplitzip.so (HIP kernels + C ABI) for gfx950 with hipcc, and the extension module _fastcall, the
binding's short way into it, with g++ and the headers of this Python and this torch.  The library works without the module."""
from __future__ import annotations

import os
import subprocess
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "csrc", "splitzip.hip")
INC = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libsplitzip.so")
FAST_SRC = os.path.join(HERE, "csrc", "fastcall.cpp")
FAST = os.path.join(HERE, "_fastcall" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))   # another Python does not find it

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall",
    # no packed-FP32 instructions from the code generator
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def build(verbose: bool = False, extra_flags=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *extra_flags, "-I", INC, SRC, "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    try:
        build_fastcall(verbose)
    except (OSError, subprocess.CalledProcessError) as e:   # no g++, or no headers
        warnings.warn(f"_fastcall was not built ({e}): the binding's calls take the general way", RuntimeWarning)
    return LIB


def build_fastcall(verbose: bool = False) -> str:
    import torch

    for old in (FAST, os.path.join(HERE, "_fastcall.so")):   # none is better than one that was built from something else
        if os.path.exists(old):
            os.remove(old)
    at = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           f'-DBUILT_FOR_TORCH="{torch.__version__}"', f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", INC, "-I", os.path.join(at, "include"),
           "-I", os.path.join(at, "include", "torch", "csrc", "api", "include"), "-I", os.path.join(rocm, "include"),
           "-I", sysconfig.get_paths()["include"], FAST_SRC, "-o", FAST, "-L", os.path.join(at, "lib"), "-ltorch_python", "-ltorch_cpu",
           "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return FAST


if __name__ == "__main__":
    print(build(verbose=True))
