"""Compile libspmm_brick.so for gfx950 with hipcc and the module _native that calls it from Python (in-tree,
next to the sources)."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libspmm_brick.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ("api.hip", "plan_kernels.hip", "exec_kernels.hip", "exec_narrow.hip", "exec_wide.hip", "exec_bf16.hip",
           "tm32_kernels.hip", "calibrate.hip")

FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
    # hand-written kernels must not use packed fp32 ops on these machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # a kernel's leading arguments are in scalar registers when a wavefront starts
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
    "-Wall", "-Wno-unused-command-line-argument",
]


def build_library(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *FLAGS, "-o", LIB, *[os.path.join(CSRC, s) for s in SOURCES]]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


def built_for() -> str:
    """What _native is tied to, as it stands in the module."""
    import torch
    return f"_native for torch {torch.__version__}, Python {sys.version_info[0]}.{sys.version_info[1]}"


def native_is_current() -> bool:
    """_native is there, made for the torch and the Python that run (looked up in the file: to load another is too
    late)."""
    if not os.path.exists(NATIVE):
        return False
    with open(NATIVE, "rb") as f:
        return built_for().encode() + b"\0" in f.read()


def build_missing() -> None:
    """What tests and the smoke run load.  The calls of _native have a slower way round it, so not every machine needs
    to be able to compile it."""
    if not os.path.exists(LIB):
        build_library()
    if not native_is_current():
        try:
            build_native()
        except (OSError, subprocess.CalledProcessError) as e:
            warnings.warn(f"_native was not built: {e}", RuntimeWarning)


def build_native(verbose: bool = False) -> str:
    """Host code only, against the headers of the installed torch."""
    import torch
    from torch.utils import cpp_extension
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f'-DSPMM_BUILT_FOR="{built_for()}"',
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *[f for p in cpp_extension.include_paths("cuda") for f in ("-isystem", p)],
           "-isystem", sysconfig.get_paths()["include"],
           "-o", NATIVE, os.path.join(CSRC, "native.cpp"),
           "-L" + lib, "-Wl,-rpath," + lib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return NATIVE


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_native(verbose=True))
