"""Build libe3.so (HIP, gfx950) with hipcc and the binding's native calls (host only) with g++, in-tree."""
from __future__ import annotations

import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libe3.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["e3_api.hip", "vocab_pass.hip", "restricted.hip", "restricted_select.hip", "probe.hip", "advantages.hip", "objective.hip",
           "scheduler.cpp", "budget.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-fno-gpu-rdc", "-ffp-contract=on",
    # packed fp32 VALU forms are not used
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def build(verbose: bool = False, extra=()) -> str:
    cmd = [HIPCC, *FLAGS, *extra, "-o", LIB] + [os.path.join(CSRC, s) for s in SOURCES]
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
    # hipcc's host pass does not know the device-only target feature and says so once
    # per function; drop that line, keep everything else
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if err.strip():
        print(err)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed with status {res.returncode}")
    build_native(verbose)
    return LIB


def build_native(verbose: bool = False) -> str:
    # NDEBUG: otherwise the headers bring a thread-local variable (pybind11's reference counter).  While the library with
    # thread-local storage that was loaded last has not touched it, glibc (before 2.39) takes the slow way to every other
    # library's.  A vocabulary pass touches libe3.so's and ends that; with a variable here that nothing touches, each torch
    # call of the process stayed 0.3 us longer, an allocated output 1.33 instead of 1.06 us.
    import torch
    root = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-DNDEBUG", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I" + os.path.join(root, "include"), "-I" + os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-I" + sysconfig.get_paths()["include"], "-o", NATIVE, os.path.join(CSRC, "native_binding.cpp"),
           "-L" + os.path.join(root, "lib"), "-lc10", "-ltorch_cpu", "-ltorch", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    return NATIVE


if __name__ == "__main__":
    print(build(verbose=True))
