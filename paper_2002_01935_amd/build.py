"""Compile libtn.so (HIP, gfx950) and the binding's _leaves.so in-tree.

    python -m paper_2002_01935_amd.build

Every source under csrc/ is compiled with hipcc for gfx950 only.  Packed FP32
instructions are disabled for the device code (see the hipcc flags).
"""

from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtn.so")
SOURCES = ["plan.cpp", "kernels.hip", "smallk.hip", "tiny.hip", "exec.hip", "batch.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
]


def build_leaves(verbose: bool = False) -> str:
    """The binding's host extension (csrc/leaves.cpp), compiled for the host
    against the installed PyTorch's headers."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    out = os.path.join(HERE, "_leaves.so")
    # any host compiler: the one that ROCm ships where there is no other (not
    # hipcc, which would link a second HIP runtime beside PyTorch's own)
    cxx = os.environ.get("CXX") or shutil.which("g++") or os.path.join(os.path.dirname(HIPCC), "amdclang++")
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-w",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    for d in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", d]
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd += [os.path.join(CSRC, "leaves.cpp"), "-o", out + ".tmp", f"-L{lib}", "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(out + ".tmp", out)
    return out


def build(verbose: bool = False) -> str:
    build_leaves(verbose)
    objs = []
    for src in SOURCES:
        path = os.path.join(CSRC, src)
        obj = os.path.join(CSRC, src + ".o")
        lang = ["-x", "hip"] if src.endswith(".hip") else []
        cmd = [HIPCC] + FLAGS + lang + ["-c", path, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        objs.append(obj)
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    for o in objs:
        os.remove(o)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
