"""Builds libavion_attn.so (gfx950 only, hipcc) and _avion_torch.so (host C++) in-tree.  Cross-compiles without a GPU."""
from __future__ import annotations

import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libavion_attn.so")
TORCH_MODULE = os.path.join(PKG, "_avion_torch.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed fp32 VALU forms stay off for every device function
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # MFMA accumulators live in ordinary VGPRs (no AGPR copies around the softmax arithmetic)
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-Wno-unused-command-line-argument",
    # the LDS-direct loads set M0 inside inline assembly and say so in their clobber list
    "-Wno-inline-asm",
]


def sources():
    return [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if f.endswith(".hip")]


def headers():
    hs = [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if f.endswith(".h")]
    return hs + [os.path.join(ROOT, "include", "avion_attn.h")]


def is_stale() -> bool:
    def older(built, made_from):
        return not os.path.exists(built) or any(os.path.getmtime(p) > os.path.getmtime(built) for p in made_from)
    return (older(LIB, sources() + headers()) or
            older(TORCH_MODULE, [os.path.join(CSRC, "avion_torch.cpp"), os.path.join(ROOT, "include", "avion_attn.h")]))


def build_library(verbose: bool = False, extra_flags=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *extra_flags, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           "-o", LIB, *sources()]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB


def build_torch_module(verbose: bool = False) -> str:
    """The autograd front end's native calls (host C++, csrc/avion_torch.cpp), linked against the library."""
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    includes = [*cpp_extension.include_paths("cuda"), sysconfig.get_paths()["include"]]
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-w",
           "-DUSE_ROCM=1", "-D__HIP_PLATFORM_AMD__=1",   # what torch's and HIP's headers ask of a host compiler
           "-I", os.path.join(ROOT, "include"), *(a for p in includes for a in ("-isystem", p)),
           os.path.join(CSRC, "avion_torch.cpp"), "-o", TORCH_MODULE, "-L", torch_lib, "-lc10", "-lc10_hip", "-ltorch_cpu",
           "-ltorch_hip", "-ltorch", "-ltorch_python", "-L", PKG, "-lavion_attn", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return TORCH_MODULE


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_torch_module(verbose=True))
