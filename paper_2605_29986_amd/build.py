"""Builds libcfgzip.so (hand-written HIP for gfx950) with hipcc and the binding's extension with g++, in-tree."""

from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_DIR = os.path.join(HERE, "lib")
LIB_PATH = os.path.join(LIB_DIR, "libcfgzip.so")
SOURCES = ["mask.hip", "walk.hip", "classes.hip", "engine.hip", "displacement.hip", "nfa.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-Wall",
    "-Wno-unused-function",
    # packed fp32 instructions stay off for every HIP translation unit
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def find_hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found; libcfgzip.so cannot be built")


# the binding's calls of every decode step and of the pre-computation as a CPython extension: host code only, against
# torch's headers
STEPCALL_PATH = os.path.join(LIB_DIR, "cfgzip_stepcall.so")


def build_stepcall(verbose: bool = False) -> str:
    import torch
    root = os.path.dirname(torch.__file__)
    tmp = STEPCALL_PATH + ".tmp.%d" % os.getpid()
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1",
           "-DUSE_ROCM=1", "-DBUILT_FOR_TORCH=\"%s\"" % torch.__version__,
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-I", sysconfig.get_paths()["include"], "-isystem", os.path.join(root, "include"),
           "-isystem", os.path.join(rocm, "include"), "-o", tmp, os.path.join(CSRC, "stepcall.cpp"),
           "-L", os.path.join(root, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python",
           "-Wl,-rpath," + os.path.join(root, "lib")]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, STEPCALL_PATH)
    return STEPCALL_PATH


TOOL_PATH = os.path.join(LIB_DIR, "gather_rate")  # calibration tool for the walk kernels' roofline


def build(verbose: bool = False) -> str:
    os.makedirs(LIB_DIR, exist_ok=True)
    tmp = LIB_PATH + ".tmp.%d" % os.getpid()
    cmd = [find_hipcc(), *HIPCC_FLAGS, "-o", tmp] + [os.path.join(CSRC, s) for s in SOURCES]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB_PATH)
    try:
        build_stepcall(verbose)
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        # no compiler, headers or torch for it: the binding does without, but not with one that an older source left
        if os.path.exists(STEPCALL_PATH):
            os.remove(STEPCALL_PATH)
        print(f"{STEPCALL_PATH} not built ({e}): the calls that it has go through ctypes", file=sys.stderr, flush=True)
    tool_flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    tmp = TOOL_PATH + ".tmp.%d" % os.getpid()
    cmd = [find_hipcc(), *tool_flags, "-o", tmp, os.path.join(CSRC, "tools", "gather_rate.hip")]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, TOOL_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
