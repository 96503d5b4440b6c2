"""Build libdiffopt.so (the HIP library behind include/diffopt.h) for gfx950 and
_binding.so (the native half of the Python binding).

    python paper_2211_06934_amd/build.py          # compile in-tree

Run it as a file (or through __graft_entry__.build()): importing the package
loads the library, so the build must not go through the package.

The shared library lands next to this file so that it travels with the
source tree.  Extra preprocessor definitions (tile sizes, streaming loads)
can be passed as ``defines`` for tuning builds written elsewhere.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libdiffopt.so")
BINDING = os.path.join(PKG, "_binding.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# -packed-fp32-ops: keep the compiler from forming packed fp32 VALU ops.
HIPFLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Wall", "-Wno-unused-function",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(out: str = LIB, defines=(), verbose: bool = False) -> str:
    """Compile every csrc/*.hip into one shared library; returns its path."""
    tmp = out + ".tmp%d" % os.getpid()
    cmd = [HIPCC, *HIPFLAGS, "-I", INCLUDE, "-I", CSRC,
           *["-D%s" % d for d in defines], *sources(), "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed building %s" % out)
    os.replace(tmp, out)
    return out


def build_binding(out: str = BINDING, lib: str = LIB, verbose: bool = False) -> str:
    """Compile csrc/binding.cpp (the native half of the Python binding, host code
    only) against torch and the library next to it; returns its path."""
    import sysconfig

    import torch
    troot = os.path.dirname(os.path.abspath(torch.__file__))
    tlib, tinc = os.path.join(troot, "lib"), os.path.join(troot, "include")
    tmp = out + ".tmp%d" % os.getpid()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch.compiled_with_cxx11_abi()),
           "-I", INCLUDE, "-isystem", tinc, "-isystem", os.path.join(tinc, "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "binding.cpp"),
           "-L", os.path.dirname(lib), "-l:" + os.path.basename(lib), "-L", tlib, "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10",
           "-Wl,-rpath,$ORIGIN", "-Wl,-rpath," + tlib, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("g++ failed building %s" % out)
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_binding(verbose=True))
