"""Build the C-ABI HIP library (``libgss.so``) for gfx950 and the binding's CPython module (``gss_torch.so``), in-tree
next to their sources."""
from __future__ import annotations

import os
import subprocess
import sysconfig

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
LIB_PATH = os.path.join(_HERE, "libgss.so")
BINDING_PATH = os.path.join(_HERE, "gss_torch.so")
SOURCES = ["gss_kernels.hip", "gss_api.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function"]


def build_library(verbose: bool = False) -> str:
    """Compile every HIP source into ``libgss.so`` (always recompiles)."""
    cmd = [HIPCC] + FLAGS + ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    cmd += [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB_PATH]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    return LIB_PATH


def build_binding(verbose: bool = False) -> str:
    """Compile ``csrc/gss_torch.cpp`` against PyTorch's headers (host code only; always recompiles)."""
    import torch
    base = os.path.dirname(os.path.abspath(torch.__file__))
    inc, lib = os.path.join(base, "include"), os.path.join(base, "lib")
    rocm = os.path.dirname(os.path.dirname(HIPCC))
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"), "-isystem", inc,
           "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "gss_torch.cpp"), "-o", BINDING_PATH, "-L", lib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    return BINDING_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_binding(verbose=True))
