"""Builds liblantern.so (the C-ABI library of include/lantern.h) for gfx950 with hipcc, and _marshal.so, the host
half of its step calls for PyTorch (csrc/marshal.cpp, host code only).

hipcc cross-compiles without a GPU.  The libraries are built in-tree, next to
this file, so that they travel with the source tree.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
import warnings

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
LIB_PATH = os.path.join(_HERE, "liblantern.so")
MARSHAL_PATH = os.path.join(_HERE, "_marshal.so")
SOURCES = ("api.hip", "verify.hip", "greedy.hip", "chain.hip", "sequential.hip", "knn.hip", "random_table.hip", "probe.hip")

HIPCC_FLAGS = (
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # every fp operation is rounded on its own: the fp64 kernels reproduce the
    # written formulas operation by operation
    "-ffp-contract=off",
    # no packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
)


def hipcc_path() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def marshal_built_for() -> str:
    """What _marshal.so depends on: it is taken by the same PyTorch and Python alone."""
    return "PyTorch %s, Python %d.%d" % (torch.__version__, *sys.version_info[:2])


def marshal_command() -> list:
    """Host code against PyTorch's C++ interface: by the host compiler, whose names PyTorch's libraries carry."""
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc_path())))
    home = os.path.dirname(torch.__file__)
    abi = int(torch._C._GLIBCXX_USE_CXX11_ABI)
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
            f"-D_GLIBCXX_USE_CXX11_ABI={abi}", f'-DLANTERN_BUILT_FOR="{marshal_built_for()}"', "-isystem", os.path.join(home, "include"),
            "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(rocm, "include"),
            "-I", os.path.join(_ROOT, "include"),
            os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL_PATH, "-L", os.path.join(home, "lib"),
            "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


def build(verbose: bool = False) -> str:
    """Compiles every source to an object (in parallel, in a scratch directory) and links the libraries.  Where _marshal.so
    cannot be built (it takes a host compiler and the headers of Python and PyTorch) there is none, and a warning."""
    import concurrent.futures
    import tempfile

    flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    inc = ["-I", os.path.join(_ROOT, "include"), "-I", CSRC]
    with tempfile.TemporaryDirectory(prefix="lantern_build_") as tmp:
        def compile_one(name: str) -> str:
            obj = os.path.join(tmp, os.path.splitext(name)[0] + ".o")
            cmd = [hipcc_path(), *flags, *inc, "-c", os.path.join(CSRC, name), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj

        def marshal() -> None:
            if verbose:
                print(" ".join(marshal_command()), flush=True)
            if os.path.exists(MARSHAL_PATH):
                os.remove(MARSHAL_PATH)
            try:
                subprocess.run(marshal_command(), check=True)
            except (OSError, subprocess.CalledProcessError) as e:
                warnings.warn(f"{MARSHAL_PATH} could not be built: {e}", RuntimeWarning)

        with concurrent.futures.ThreadPoolExecutor(max_workers=min(len(SOURCES) + 1, os.cpu_count() or 1, 8)) as pool:
            host = pool.submit(marshal)
            objs = list(pool.map(compile_one, SOURCES))
            host.result()
        link = [hipcc_path(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs]
        if verbose:
            print(" ".join(link), flush=True)
        subprocess.run(link, check=True)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
