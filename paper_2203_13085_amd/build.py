"""Compile the HIP library in-tree for gfx950 (cross-compiles without a GPU), and the host extension of the torch class."""
from __future__ import annotations

import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "lasgd.hip")
LIB = os.path.join(HERE, "liblasgd_hip.so")
WALK_SRC = os.path.join(HERE, "csrc", "grad_walk.cpp")
WALK_LIB = os.path.join(HERE, "_grad_walk" + sysconfig.get_config_var("EXT_SUFFIX"))     # another Python does not load it

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17",
    "-ffp-contract=off",                      # only the written fmaf calls fuse
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-fPIC", "-shared", "-Wall", "-Wno-unused-function",
]


def build_hip(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + FLAGS + ["-o", LIB, SRC]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


def build_grad_walk(verbose: bool = False) -> str:
    """Host code against the installed torch's headers and libraries."""
    import torch
    root = os.path.dirname(torch.__file__)
    inc = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
           sysconfig.get_paths()["include"]]
    lib = os.path.join(root, "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DLASGD_TORCH_VERSION="{torch.__version__}"', *["-isystem" + d for d in inc], "-o", WALK_LIB, WALK_SRC, "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10",
           "-Wl,-rpath," + lib]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return WALK_LIB


if __name__ == "__main__":
    print(build_hip(verbose=True))
    print(build_grad_walk(verbose=True))
