"""Ahead-of-time build of libdvgo.so for gfx950 with hipcc, and of the C++ autograd nodes that call it
(_dvgo_autograd.so, a Python extension on libtorch) with the host compiler (no JIT)."""
from __future__ import annotations

import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libdvgo.so")
NATIVE = os.path.join(HERE, "_dvgo_autograd.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# -packed-fp32-ops: no v_pk_*_f32 generation (kept scalar on purpose).
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))


def build_autograd(verbose: bool = False) -> str:
    """The C++ autograd nodes (csrc/autograd.cpp); needs libdvgo.so beside it."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    tmp = NATIVE + ".tmp"
    rocm = os.path.dirname(os.path.dirname(HIPCC))
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    inc = [*cpp_extension.include_paths(), sysconfig.get_paths()["include"], os.path.join(rocm, "include"),
           os.path.join(ROOT, "include")]
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-fvisibility=hidden",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-DTORCH_API_INCLUDE_EXTENSION_H",
           f"-DTORCH_EXTENSION_NAME={os.path.basename(NATIVE)[:-3]}",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *[a for i in inc for a in ("-isystem", i)], os.path.join(HERE, "csrc", "autograd.cpp"), "-o", tmp,
           "-L" + libs, "-ltorch", "-ltorch_cpu", "-ltorch_hip", "-lc10", "-lc10_hip", "-ltorch_python",
           "-L" + HERE, "-l:libdvgo.so", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, NATIVE)
    return NATIVE


def build(verbose: bool = False) -> str:
    srcs = sources()
    tmp = LIB + ".tmp"
    cmd = [HIPCC, *FLAGS, "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc"), "-o", tmp, *srcs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    try:
        build_autograd(verbose)
    except (subprocess.CalledProcessError, OSError) as e:
        # no host C++ compiler, or one that does not take this libtorch's headers: the package works without
        # the nodes, and an older build of them does not belong to this library
        if os.path.exists(NATIVE):
            os.remove(NATIVE)
        print(f"warning: the C++ autograd nodes were not built ({e}); the Python Functions take their place",
              file=sys.stderr, flush=True)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    print(LIB)
    sys.exit(0)
