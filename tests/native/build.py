"""Builds the native test programs (test infrastructure; __graft_entry__.build()
calls build() after the library):

  abi_driver  a plain C++ program that uses libdisdp.so through
              include/disdp.h with the system HIP runtime and no PyTorch;
  api_fuzz    the C-ABI front end (disdp_api.cpp) compiled with g++ under
              AddressSanitizer and UndefinedBehaviorSanitizer, host code
              only, with stub HIP calls, fuzzed without a GPU;
  launch_check
              the host code of the kernels' file, with stub HIP calls, its
              launches checked without a GPU."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
SRC = os.path.join(HERE, "abi_driver.cpp")
EXE = os.path.join(HERE, "abi_driver")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
PKG = os.path.join(ROOT, "paper_2409_00918_amd")


FUZZ_SRC = os.path.join(HERE, "api_fuzz.cpp")
FUZZ_EXE = os.path.join(HERE, "api_fuzz")
API_SRC = os.path.join(PKG, "csrc", "disdp_api.cpp")


def build_fuzz(verbose: bool = False) -> str:
    """g++ (host code only, no HIP device code) with both sanitizers."""
    tmp = FUZZ_EXE + ".tmp"
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-Wall",
           "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
           "-o", tmp, FUZZ_SRC, API_SRC]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, FUZZ_EXE)
    return FUZZ_EXE


LAUNCH_SRC = os.path.join(HERE, "launch_check.cpp")
LAUNCH_EXE = os.path.join(HERE, "launch_check")


def build_launch_check(verbose: bool = False) -> str:
    """Host code only, linked without the HIP runtime (its calls are stubs)."""
    obj, tmp = LAUNCH_EXE + ".o", LAUNCH_EXE + ".tmp"
    cmds = [[HIPCC, "-std=c++17", "-O1", "-fPIC", "-Wall", "-Wno-unused-function",
             "-Wno-unused-command-line-argument", "-x", "hip", "--offload-arch=gfx950",
             "--cuda-host-only", "-fuse-cuid=none", "-I", os.path.join(ROOT, "include"),
             "-I", os.path.join(PKG, "csrc"), "-c", "-o", obj, LAUNCH_SRC],
            ["g++", "-o", tmp, obj]]
    for cmd in cmds:
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
    os.remove(obj)
    os.replace(tmp, LAUNCH_EXE)
    return LAUNCH_EXE


def build(verbose: bool = False) -> str:
    tmp = EXE + ".tmp"
    cmd = [HIPCC, "-O2", "-std=c++17", "-Wall", "-Wno-unused-command-line-argument",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "include"), "-o", tmp, SRC,
           "-L", PKG, "-ldisdp", "-Wl,-rpath,$ORIGIN/../../paper_2409_00918_amd", "-ldl"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, EXE)
    build_fuzz(verbose)
    build_launch_check(verbose)
    return EXE


if __name__ == "__main__":
    print(build(verbose=True))
