"""Builds libppv_hip.so (the C-ABI library) for gfx950 with hipcc, and _ppv_call.so (the Python side's native calls), in-tree."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libppv_hip.so")
CALL = os.path.join(PKG, "_ppv_call.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed fp32 instructions stay off for every kernel of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # no multiply-add fusing beyond the fmaf calls in the sources: several kernels promise each other's results bit
    # for bit, which must not hinge on where the compiler happens to find a multiply next to an add
    "-ffp-contract=off",
    # a kernel's leading scalar arguments arrive in registers (the kernels take first what their first loads need)
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(verbose: bool = True) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", LIB, *sources()]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    build_call(verbose)
    return LIB


def build_call(verbose: bool = True) -> str:
    """The CPython extension of binding.py: host code only, against torch's headers and libraries."""
    import torch
    at = os.path.dirname(torch.__file__)
    include = [os.path.join(ROOT, "include"), os.path.join(at, "include"),
               os.path.join(at, "include", "torch", "csrc", "api", "include"),
               os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), sysconfig.get_path("include")]
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1",
           "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", include[0], *[x for d in include[1:] for x in ("-isystem", d)], os.path.join(CSRC, "ppv_call.cpp"),
           "-o", CALL, "-L", os.path.join(at, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return CALL


if __name__ == "__main__":
    build()
    sys.exit(0)
