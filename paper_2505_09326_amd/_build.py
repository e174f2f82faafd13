"""Compile the HIP library for gfx950 (in-tree, so the .so travels with the source tree)."""
from __future__ import annotations

import os
import subprocess

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB_PATH = os.path.join(_HERE, "libsphattn.so")
MARSHAL_PATH = os.path.join(_HERE, "_marshal.so")
SOURCES = [os.path.join(CSRC, "sphattn_api.hip")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # keep hipcc from forming packed-fp32 VALU instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # select matrix-core instructions in their VGPR-destination form and let the register
    # allocator move long-lived accumulators/operands to AGPRs; without it every MFMA result
    # lands in AGPRs and the score registers must be copied out before the VALU can touch them
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    # Tile loops begin on an instruction cache line.  One wave per SIMD has nothing to cover the fetch behind the
    # branch back, so where a loop happens to land counts: the d = 128 forward 4 bytes before the end of a line
    # took 60 cycles more per tile (9 x 8192 x 128 272.8 us, 3 x 25243 x 128 811) than in the middle of one or at
    # its start (265 and 790).
    "-falign-loops=64",
    "-Wno-unused-command-line-argument",
]


def build_library(verbose: bool = False) -> str:
    """Run hipcc unconditionally and return the path of the shared library."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, "-o", LIB_PATH, *SOURCES]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if verbose or res.returncode != 0:
        print(" ".join(cmd))
        print(res.stdout)
        print(res.stderr)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed building libsphattn.so")
    return LIB_PATH


def build_marshal(verbose: bool = False) -> str:
    """Compile the CPython extension in front of the library (csrc/marshal.cpp; host code only) and return its path."""
    import sysconfig
    import torch
    base = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DMARSHAL_TORCH="{torch.__version__}"',
           f"-I{base}/include", f"-I{base}/include/torch/csrc/api/include", "-I/opt/rocm/include", f"-I{sysconfig.get_paths()['include']}",
           "-o", MARSHAL_PATH, os.path.join(CSRC, "marshal.cpp"), f"-L{base}/lib", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if verbose or res.returncode != 0:
        print(" ".join(cmd))
        print(res.stdout)
        print(res.stderr)
    if res.returncode != 0:
        raise RuntimeError("the compiler failed building _marshal.so")
    return MARSHAL_PATH
