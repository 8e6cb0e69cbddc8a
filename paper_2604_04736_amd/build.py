"""Compiles csrc/*.hip into libhot.so (hipcc, gfx950 only) and csrc/host_ops.cpp into _hot_host.so (host code), next to this file."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRCS = [os.path.join(HERE, "csrc", name) for name in ("forward.hip", "backward.hip", "hot.hip", "stats.hip", "linear.hip", "update.hip")]
LIB = os.path.join(HERE, "libhot.so")
HOST_LIB = os.path.join(HERE, "_hot_host.so")
OBJ_DIR = os.path.join(HERE, "_build")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# Packed fp32 arithmetic is switched off for all device code of this library.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-I", os.path.join(ROOT, "include")]


def _run(cmd, verbose):
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if verbose or res.returncode != 0:
        sys.stderr.write(res.stdout)
    if res.returncode != 0:
        raise RuntimeError("the compiler failed building libhot.so or _hot_host.so: " + " ".join(cmd[-3:]))


def build_libhot(verbose: bool = False) -> str:
    """One object per source file, compiled side by side, then one link."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    objs = [os.path.join(OBJ_DIR, os.path.basename(src) + ".o") for src in SRCS]
    with ThreadPoolExecutor(max_workers=len(SRCS)) as pool:
        list(pool.map(lambda so: _run([HIPCC] + FLAGS + ["-c", "-o", so[1], so[0]], verbose), zip(SRCS, objs)))
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs, verbose)
    build_host_ops(verbose)
    return LIB


def build_host_ops(verbose: bool = False) -> str:
    """The Python module around libhot.so's calls (torch's C++ interface; no device code)."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    includes = cpp_extension.include_paths() + [sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
          f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *("-I" + p for p in includes), "-o", HOST_LIB,
          os.path.join(HERE, "csrc", "host_ops.cpp"), "-L" + HERE, "-lhot", "-Wl,-rpath,$ORIGIN", "-L" + torch_lib, "-lc10",
          "-ltorch_cpu", "-ltorch_python", "-Wl,-rpath," + torch_lib], verbose)
    return HOST_LIB


if __name__ == "__main__":
    print(build_libhot(verbose=True))
