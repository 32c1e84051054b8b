"""Build libanszp.so in-tree with hipcc for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libanszp.so")
SOURCES = [os.path.join(CSRC, "anszp_host.cpp"), os.path.join(CSRC, "anszp_device.hip"),
           os.path.join(CSRC, "anszp_conv.hip"), os.path.join(CSRC, "anszp_encode.hip")]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include")]


TEST_HELPER_SRC = os.path.join(ROOT, "tests", "gpu_helpers", "lds_fill.hip")
TEST_HELPER_LIB = os.path.join(ROOT, "tests", "gpu_helpers", "liblds_fill.so")


def build_test_helpers(verbose: bool = False) -> str:
    """The GPU tests' own helper kernels (tests/gpu_helpers), built in-tree like the library."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-o", TEST_HELPER_LIB, TEST_HELPER_SRC]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return TEST_HELPER_LIB


HOST_SRC = os.path.join(CSRC, "anszp_torch.cpp")
HOST_LIB = os.path.join(HERE, "_anszp_torch.so")


def build_host_calls(verbose: bool = False) -> str:
    """The binding's native calls (host code, against torch's headers and the library), in-tree like the library."""
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", os.path.join(ROOT, "include"), *[f for d in include_paths() + [sysconfig.get_paths()["include"]] for f in ("-isystem", d)],
           "-o", HOST_LIB, HOST_SRC, "-L", HERE, "-l:" + os.path.basename(LIB), "-L", lib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return HOST_LIB


def build_library(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + FLAGS + ["-o", LIB] + SOURCES
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_host_calls(verbose=True))
    print(build_test_helpers(verbose=True))
