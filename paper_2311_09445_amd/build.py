"""Builds libper_hip.so (gfx950) and the Python boundary of its per-iteration calls in-tree.  Usable as
``python -m paper_2311_09445_amd.build``."""
from __future__ import annotations

import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libper_hip.so")
BINDING = os.path.join(HERE, "_per_binding.so")
SOURCES = ["per_kernels.hip", "per_api.hip"]

# -ffp-contract=off: the tree arithmetic must round after every add and multiply.
# packed-fp32 ops are switched off for the device pass.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
         "-fno-fast-math", "-fno-gpu-flush-denormals-to-zero",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-command-line-argument"]


def build_lib(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + [f for f in FLAGS if f] + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


def build_binding(verbose: bool = False) -> str:
    """Host code only (no kernels): the CPython module that takes torch tensors apart for the C-ABI calls."""
    from torch.utils import cpp_extension
    torch_lib = os.path.join(os.path.dirname(cpp_extension.include_paths()[0]), "lib")
    include = cpp_extension.include_paths() + ["/opt/rocm/include", sysconfig.get_paths()["include"]]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1"]
    cmd += [x for d in include for x in ("-isystem", d)] + [os.path.join(CSRC, "per_binding.cpp"), "-o", BINDING]
    cmd += ["-L" + HERE, "-l:libper_hip.so", "-Wl,-rpath,$ORIGIN", "-L" + torch_lib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return BINDING


if __name__ == "__main__":
    print(build_lib(verbose=True))
    print(build_binding(verbose=True))
