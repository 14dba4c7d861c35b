"""Builds libdynadiag.so (the HIP kernels plus the C ABI) for gfx950 with hipcc and _fastcall.so (the binding's short way to it),
in-tree."""
import glob
import os
import subprocess
import sysconfig

import torch

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libdynadiag.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-Wall",
    "-Wno-unused-command-line-argument",
    # packed fp32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build_library(verbose=False):
    """Compile every csrc/*.hip into one shared library.  Always recompiles."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, "-o", LIB_PATH, *sources()]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    build_fastcall(verbose)
    return LIB_PATH


FASTCALL_SRC = os.path.join(CSRC, "fastcall.cpp")
FASTCALL_PATH = os.path.join(PKG_DIR, "_fastcall.so")


def build_fastcall(verbose=False):
    """Compile the Python extension (host code against torch's headers, no device code)."""
    root = os.path.dirname(os.path.abspath(torch.__file__))
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(root, "include"), "-o", FASTCALL_PATH, FASTCALL_SRC,
           "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return FASTCALL_PATH


CEILINGS_SRC = os.path.join(PKG_DIR, "ceilings", "ceilings.hip")
CEILINGS_BIN = os.path.join(PKG_DIR, "ceilings", "ceilings")


def build_ceilings():
    """Compile the stand-alone ceilings microbenchmark (not part of the library)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                           "-o", CEILINGS_BIN, CEILINGS_SRC])
    return CEILINGS_BIN


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_ceilings())
