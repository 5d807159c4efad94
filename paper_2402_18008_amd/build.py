"""Build libhomog.so (HIP, gfx950) and the binding's native call path
(_native.so, host code against torch's headers) next to this file.

Usage: python -m paper_2402_18008_amd.build   (or build() from Python)
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhomog.so")
NATIVE = os.path.join(HERE, "_native.so")

SOURCES = ["status.hip", "solve.hip", "ransac.hip", "diff.hip", "refit.hip", "stream.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    # every rounding is the one written in the source (no implicit contraction)
    "-ffp-contract=off",
    # no packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def _run(cmd, what, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"{cmd[0]} failed building {what}")


def build_native(verbose=False):
    """_native.so: the host compiler, torch's headers and libraries; it finds
    libhomog.so beside itself. It is optional (without it every call goes through
    ctypes), so where there is no compiler or a header is missing it is left out,
    with a message, and one that was built before, against another libhomog, goes:
    returns None then."""
    import torch
    root = os.path.dirname(torch.__file__)
    python = sysconfig.get_paths()["include"]
    cxx = shutil.which("g++") or shutil.which("c++")
    needed = [os.path.join(root, "include", "torch", "csrc", "autograd", "python_variable.h"),
              os.path.join(python, "Python.h")]
    missing = [] if cxx else ["a C++ compiler"]
    missing += [h for h in needed if not os.path.exists(h)]
    if missing:
        sys.stderr.write(f"_native.so is not built: {', '.join(missing)} not found\n")
        if os.path.exists(NATIVE):
            os.remove(NATIVE)
        return None
    inc = [os.path.join(ROOT, "include"), os.path.join(root, "include"),
           os.path.join(root, "include", "torch", "csrc", "api", "include"),
           os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), python]
    tmp = NATIVE + ".tmp"
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-w",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *(f for i in inc for f in ("-isystem", i)), "-o", tmp,
           os.path.join(CSRC, "binding.cpp"), LIB, "-L", os.path.join(root, "lib"),
           "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-Wl,-rpath,$ORIGIN"]
    _run(cmd, "_native.so", verbose)
    os.replace(tmp, NATIVE)
    return NATIVE


def build(verbose=False):
    srcs = [os.path.join(CSRC, s) for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    tmp = LIB + ".tmp"
    cmd = [hipcc(), *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", tmp, "-Wl,-soname,libhomog.so", *srcs]
    _run(cmd, "libhomog.so", verbose)
    os.replace(tmp, LIB)
    build_native(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
