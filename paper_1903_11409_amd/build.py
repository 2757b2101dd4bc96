"""Builds libbspmm.so (HIP kernels + scheduler + C ABI) for gfx950 with hipcc, and _native.so (the
CPython side of the binding) beside it, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbspmm.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["kernels.hip", "schedule.cpp", "api.cpp", "staging.cpp"]
NATIVE_SOURCES = ["binding.cpp"]
HEADERS = ["plan.hpp", "schedule.hpp", "plan_api.hpp", "staging.hpp", os.path.join("..", "..", "include", "bspmm.h")]


def lib_path() -> str:
    return LIB


def is_stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(NATIVE):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(NATIVE))
    return any(os.path.getmtime(os.path.join(CSRC, f)) > t for f in SOURCES + NATIVE_SOURCES + HEADERS)


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError(os.path.basename(cmd[0]) + " failed:\n" + r.stdout)
    if verbose and r.stdout.strip():
        print(r.stdout, file=sys.stderr)


def build_library(verbose: bool = False) -> str:
    """Compile every source for gfx950 and link libbspmm.so, which needs neither PyTorch nor numpy.  Always
    recompiles."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           # kernels whose arguments are plain pointers and integers get them in SGPRs when a
           # wavefront starts (the command processor fills up to 16 of them): their first
           # dependent fetch, the work item, goes out at once instead of after a kernel-argument
           # load
           "-mllvm", "-amdgpu-kernarg-preload-count=16",
           "-Wall", "-Wno-unused-command-line-argument", "-Wno-inline-asm",
           "-x", "hip", os.path.join(CSRC, "kernels.hip"),
           "-x", "hip", os.path.join(CSRC, "schedule.cpp"),
           "-x", "hip", os.path.join(CSRC, "api.cpp"),
           "-x", "hip", os.path.join(CSRC, "staging.cpp"),
           "-o", LIB]
    _run(cmd, verbose)
    return LIB


def build(verbose: bool = False) -> str:
    """The library, then the extension module that binds it to PyTorch.  Always recompiles."""
    build_library(verbose)
    # the extension module finds libbspmm.so in its own folder; PyTorch's libraries are loaded before it
    import numpy
    import torch
    root = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    native = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
              "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
              "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
              "-I" + sysconfig.get_paths()["include"], "-isystem", numpy.get_include(),
              "-isystem", os.path.join(root, "include"),
              "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
              "-isystem", os.path.join(rocm, "include"), os.path.join(CSRC, "binding.cpp"),
              "-L" + HERE, "-l:libbspmm.so", "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu",
              "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN", "-o", NATIVE]
    _run(native, verbose)
    return LIB


if __name__ == "__main__":
    print((build_library if sys.argv[1:] == ["library"] else build)(verbose=True))
