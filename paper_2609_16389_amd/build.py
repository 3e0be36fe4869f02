"""Build libxgemm.so (the HIP library behind include/xgemm.h) for gfx950 and
_fastcall.so (its calls from Python), in-tree."""
from __future__ import annotations

import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SRC = os.path.join(PKG, "csrc", "xgemm.hip")
DEPS = [SRC, os.path.join(PKG, "csrc", "direct_kernel.hpp"), os.path.join(PKG, "csrc", "gemm_kernel.hpp"), os.path.join(PKG, "csrc", "gemv_kernel.hpp"),
        os.path.join(PKG, "csrc", "pack_kernel.hpp"), os.path.join(PKG, "csrc", "sk_kernel.hpp"),
        os.path.join(ROOT, "include", "xgemm.h")]
LIB = os.path.join(PKG, "libxgemm.so")
FAST_SRC = os.path.join(PKG, "csrc", "fastcall.cpp")
FAST_LIB = os.path.join(PKG, "_fastcall.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# Packed fp32 vector ops are disabled for all device code.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++20", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(ROOT, "include")]


def build(verbose: bool = False) -> str:
    """Compile the library; always rebuilds.  Returns the path of the .so."""
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [HIPCC] + FLAGS + [SRC, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    build_fastcall(verbose)
    return LIB


def fastcall_tag() -> str:
    """What the extension has to be built for: it reads torch's tensors by
    their C++ layout."""
    import sys

    import torch
    return "xgemm fastcall, Python %d.%d, torch %s" % (sys.version_info[0], sys.version_info[1], torch.__version__)


def fastcall_is_current() -> bool:
    """Whether the extension is there and built for this Python and torch."""
    if not os.path.exists(FAST_LIB):
        return False
    with open(FAST_LIB, "rb") as f:
        return fastcall_tag().encode() + b"\0" in f.read()


def build_fastcall(verbose: bool = False) -> str:
    """Compile the Python extension against Python's and torch's headers (host
    code only)."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    tmp = FAST_LIB + ".tmp%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1",
           "-DUSE_ROCM=1", '-DXGEMM_FASTCALL_TAG="%s"' % fastcall_tag(), "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           "-I" + os.path.join(root, "include"), "-I" + os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-I" + sysconfig.get_paths()["include"], "-I/opt/rocm/include", FAST_SRC, "-o", tmp,
           "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, FAST_LIB)
    return FAST_LIB


def is_stale() -> bool:
    if not os.path.exists(LIB) or not fastcall_is_current():
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(d) > t for d in DEPS) or os.path.getmtime(FAST_SRC) > os.path.getmtime(FAST_LIB)


if __name__ == "__main__":
    print(build(verbose=True))
