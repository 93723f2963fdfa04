"""Builds libhp.so (the C-ABI library: host plan builder + gfx950 kernels) with
hipcc and hp_marshal.so (the binding's tensor marshalling) with g++, in-tree,
next to the sources' package."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from typing import Optional

_PKG = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_PKG)
CSRC = os.path.join(_PKG, "csrc")
LIB_PATH = os.path.join(_PKG, "libhp.so")
SOURCES = ["hp_api.hip", "hp_plan.cpp"]
MARSHAL_PATH = os.path.join(_PKG, "hp_marshal.so")

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared",
    "--offload-arch=gfx950",
    # keep hipcc from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the backward fold is a fixed-order chain of plain binary32 adds
    "-ffp-contract=off", "-fno-fast-math",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
]


def hipcc_path() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the HIP library cannot be built on this machine")


def build_marshal(verbose: bool = False) -> Optional[str]:
    """Compile the CPython extension that takes torch tensors to the C ABI.  The
    library and its binding do without it (the binding's calls are then some
    microseconds slower): where torch, its headers or g++ are missing this
    says so, leaves no older one behind, and returns None."""
    import sysconfig
    if os.path.exists(MARSHAL_PATH):
        os.remove(MARSHAL_PATH)
    try:
        import torch
    except ImportError:
        print("hp_marshal.so not built: torch is not installed", file=sys.stderr, flush=True)
        return None
    t = os.path.dirname(torch.__file__)
    cmd = ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Wextra", "-Wno-unused-parameter",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DHP_TORCH_VERSION="{torch.__version__}"',
           "-I", os.path.join(_ROOT, "include"), "-isystem", sysconfig.get_paths()["include"],
           "-isystem", os.path.join(t, "include"), "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"),
           "-o", MARSHAL_PATH, os.path.join(CSRC, "hp_marshal.cpp"),
           "-L" + os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        res = subprocess.run(cmd, capture_output=True, text=True)
    except OSError as e:
        print(f"hp_marshal.so not built: {e}", file=sys.stderr, flush=True)
        return None
    if res.returncode != 0:
        print("hp_marshal.so not built: g++ failed:\n" + res.stdout + res.stderr, file=sys.stderr, flush=True)
        return None
    return MARSHAL_PATH


def build_library(verbose: bool = False, extra_flags=()) -> str:
    """Compile every source for gfx950 into paper_2605_27678_amd/libhp.so, and
    the marshalling extension beside it where that can be built."""
    build_marshal(verbose)
    cmd = [hipcc_path(), *HIPCC_FLAGS, *extra_flags,
           "-I", os.path.join(_ROOT, "include"), "-I", CSRC,
           "-o", LIB_PATH, *[os.path.join(CSRC, s) for s in SOURCES]]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    if verbose and res.stderr.strip():
        print(res.stderr)
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
