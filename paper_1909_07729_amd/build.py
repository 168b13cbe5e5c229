"""Builds libktanh.so (the C-ABI library with the gfx950 kernels) in-tree with hipcc, and next to it
_ktanh_torch.so (host code: calls of that library on torch tensors) with the host compiler."""
from __future__ import annotations

import os
import subprocess
import sysconfig

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
LIB_PATH = os.path.join(_HERE, "libktanh.so")
SOURCES = ["ktanh_stream.hip", "ktanh_lstm.hip", "ktanh_lstm_chunks.hip", "ktanh_lstm_ring.hip",
           "ktanh_backward.hip", "ktanh_lut.cpp", "ktanh_fit.cpp"]
# measurement yardsticks (include/ktanh_probe.h): a library of their own, loaded only by the benchmark
PROBE_LIB_PATH = os.path.join(_HERE, "libktanh_probe.so")
PROBE_SOURCES = ["ktanh_probe.hip", "ktanh_lut.cpp", "ktanh_fit.cpp"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-std=c++17", "-O3", "-fPIC", "-shared",
    "-ffp-contract=off",                       # every fused multiply-add in the kernels is explicit
    "-fno-gpu-flush-denormals-to-zero",        # Float32 subnormals are kept
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the leading scalar arguments of every kernel arrive preloaded in scalar registers, so a
    # wavefront can issue its first load without a round trip to the argument buffer
    "-mllvm", "-amdgpu-kernarg-preload-count=12",
    "-Wall", "-Wextra", "-Wno-unused-command-line-argument",
]


def _compile(sources, target, verbose):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           *[os.path.join(CSRC, s) for s in sources], "-o", target]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    return target


def build_library(verbose: bool = False) -> str:
    """Compile every source of the library for gfx950; returns the path of the .so."""
    return _compile(SOURCES, LIB_PATH, verbose)


def build_probe_library(verbose: bool = False) -> str:
    """Compile the measurement yardsticks (libktanh_probe.so) for gfx950."""
    return _compile(PROBE_SOURCES, PROBE_LIB_PATH, verbose)


HOST_PATH = os.path.join(_HERE, "_ktanh_torch.so")


def build_host_path(verbose: bool = False) -> str:
    """Compile the host path of calls on torch tensors; links libktanh.so, which it finds next to itself."""
    import torch
    from torch.utils.cpp_extension import include_paths
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    includes = [*include_paths(), os.path.join(rocm, "include"), sysconfig.get_path("include")]
    cmd = [os.environ.get("CXX", "g++"), "-std=c++17", "-O2", "-fPIC", "-shared", "-Wall", "-Wextra",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f'-DKTANH_TORCH_VERSION="{torch.__version__}"',
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *[a for path in includes for a in ("-isystem", path)], "-I", os.path.join(ROOT, "include"),
           os.path.join(CSRC, "ktanh_torch.cpp"), "-o", HOST_PATH, "-L", _HERE, "-lktanh",
           "-L", torch_lib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    return HOST_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_host_path(verbose=True))
    print(build_probe_library(verbose=True))
