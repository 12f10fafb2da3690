"""Compile the HIP library libpda.so for gfx950 and the binding's native
marshalling (pda_native.so), both in-tree.

Run as ``python -m paper_2606_07665_amd.build`` or through
``__graft_entry__.build()``.  hipcc cross-compiles without a GPU.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB_DIR = os.path.join(PKG, "_lib")
LIB_PATH = os.path.join(LIB_DIR, "libpda.so")
NATIVE_PATH = os.path.join(LIB_DIR, "pda_native.so")
SOURCES = [os.path.join(CSRC, f) for f in ("pda_kernels.hip", "pda_append.hip", "pda_gemv.hip", "pda_probe.hip", "pda_scratch.hip", "pda_api.cpp")]
NATIVE_SOURCE = os.path.join(CSRC, "pda_native.cpp")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.environ.get("CXX", "g++")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Wall", "-Wno-unused-function",
    # never let the compiler form packed fp32 VALU ops (v_pk_*_f32)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed with exit code {res.returncode}")


def build_library(verbose: bool = False, extra_flags=None) -> str:
    os.makedirs(LIB_DIR, exist_ok=True)
    tmp = LIB_PATH + ".tmp"
    _run([HIPCC, *FLAGS, *(extra_flags or []), "-o", tmp, *SOURCES], verbose)
    os.replace(tmp, LIB_PATH)
    return LIB_PATH


def build_native(verbose: bool = False) -> str:
    """The CPython extension, against torch's headers (host code only); it
    carries the versions it was built for, which the binding compares."""
    import torch
    from torch.utils import cpp_extension

    from paper_2606_07665_amd.binding import _built_for
    os.makedirs(LIB_DIR, exist_ok=True)
    tmp = NATIVE_PATH + ".tmp"
    cmd = [CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DPDA_BUILT_FOR="{_built_for()}"', "-I", os.path.join(ROOT, "include"), "-I", sysconfig.get_paths()["include"]]
    for path in cpp_extension.include_paths():
        cmd += ["-isystem", path]
    cmd += ["-o", tmp, NATIVE_SOURCE]
    for path in cpp_extension.library_paths():
        cmd += ["-L", path]
    cmd += ["-ltorch_python", "-ltorch_cpu", "-lc10"]
    _run(cmd, verbose)
    os.replace(tmp, NATIVE_PATH)
    return NATIVE_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_native(verbose=True))
