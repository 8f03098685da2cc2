"""Compiles the HIP sources under csrc/ into paper_2512_23858_amd/libygg.so for gfx950, and the native half of the Python
binding (csrc/python_calls.cpp, host code only) into paper_2512_23858_amd/_calls.so."""
from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess

_PKG = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_PKG)
_CSRC = os.path.join(_PKG, "csrc")
_OBJ = os.path.join(_PKG, "_build")
LIB_PATH = os.path.join(_PKG, "libygg.so")
CALLS_PATH = os.path.join(_PKG, "_calls.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    # packed-fp32 VALU forms are kept off for every device translation unit
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option",
    "-I", os.path.join(_ROOT, "include"), "-I", _CSRC,
]


def _compile(src: str) -> str:
    obj = os.path.join(_OBJ, os.path.basename(src) + ".o")
    subprocess.check_call([HIPCC, *FLAGS, "-c", src, "-o", obj])
    return obj


def _build_calls() -> None:
    """The Python binding's native half: plain C++ against Python's and torch's headers, linked with libygg.so."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    inc = [sysconfig.get_paths()["include"], os.path.join(_ROOT, "include"), *cpp_extension.include_paths("cuda")]
    libs = cpp_extension.library_paths("cuda")
    subprocess.check_call([
        "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
        f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *(f"-I{d}" for d in inc),
        os.path.join(_CSRC, "python_calls.cpp"), "-o", CALLS_PATH, f"-L{_PKG}", "-lygg", *(f"-L{d}" for d in libs),
        "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-Wl,-rpath,$ORIGIN"])


def build(verbose: bool = False) -> str:
    """Always recompiles every source (seconds each) and relinks the shared library."""
    os.makedirs(_OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(_CSRC, "*.hip")))
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs])
    _build_calls()
    if verbose:
        print("built", LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True)
