"""Builds libmosaicattn.so for gfx950 with hipcc, in-tree (paper_2312_17482_amd/lib/)."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIBDIR = os.path.join(PKG, "lib")
LIB = os.path.join(LIBDIR, "libmosaicattn.so")
MARSHAL = os.path.join(LIBDIR, "_mosaic_marshal.so")   # Python module: host code of the binding's hot calls

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",     # no packed-fp32 VALU instructions
    "-Wall", "-Wno-unused-function", "-Wno-unknown-attributes",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


def marshal_command():
    """The compile line of csrc/marshal.cpp (plain C++ against the headers of Python and of the installed torch)."""
    import torch
    base = os.path.join(os.path.dirname(torch.__file__))
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
            "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
            "-isystem", os.path.join(base, "include"),
            "-isystem", os.path.join(base, "include", "torch", "csrc", "api", "include"),
            "-I" + sysconfig.get_paths()["include"], "-I" + os.path.join(ROOT, "include"),
            os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL,
            "-L" + os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10"]


def build(verbose: bool = True, jobs: int = 8) -> str:
    """Compile every csrc/*.hip and link the shared library, and compile the binding's native part.  Always recompiles."""
    os.makedirs(LIBDIR, exist_ok=True)
    objdir = os.path.join(LIBDIR, "obj")
    os.makedirs(objdir, exist_ok=True)
    sources = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    procs = []
    objs = []
    cmd = marshal_command()
    if verbose:
        print(" ".join(cmd), flush=True)
    procs.append((os.path.join(CSRC, "marshal.cpp"), subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src in sources:
        obj = os.path.join(objdir, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        cmd = [HIPCC] + FLAGS + ["-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        if len(procs) >= jobs:
            _drain(procs)
    _drain(procs)
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    out = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if out.returncode != 0:
        raise RuntimeError("link failed:\n" + out.stdout)
    return LIB


def _drain(procs):
    for src, p in procs:
        out, _ = p.communicate()
        # the host pass does not know the GPU-only target feature; that warning is harmless
        lines = [l for l in out.splitlines() if "packed-fp32-ops" not in l and "is not a recognized feature" not in l]
        text = "\n".join(lines).strip()
        if p.returncode != 0:
            raise RuntimeError("compiling %s failed:\n%s" % (src, out))
        if text:
            print(text, file=sys.stderr)
    procs.clear()


if __name__ == "__main__":
    print(build())
