"""Build the HIP library (gfx950) in-tree: ``python -m paper_2411_05289_amd.build``.

Every ``csrc/*.hip`` file is one kernel family (or the host side) and is compiled to an object
of its own, several at a time; the objects are then linked into ``libmdsd.so``."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmdsd.so")
HOST = os.path.join(HERE, "_host.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off",                       # fused multiply-adds only where written
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def sources():
    return [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if f.endswith(".hip")]


def jobs() -> int:
    try:
        n = int(os.environ.get("MAX_JOBS", "0"))
    except ValueError:
        n = 0
    return max(1, min(n or (os.cpu_count() or 1), 16))


def host_compiler() -> str:
    """$CXX, the system's C++ compiler, or the one that comes with hipcc."""
    names = [os.environ.get("CXX"), "g++", "c++",
             os.path.join(os.path.dirname(HIPCC), "..", "llvm", "bin", "clang++")]
    for name in names:
        found = shutil.which(name) if name else None
        if found:
            return found
    raise RuntimeError("no C++ compiler found; set CXX")


def build_host(verbose: bool = True):
    """The native marshalling of the Python binding (host code only), linked to libmdsd.so.  Left out, with a
    message, where there is no torch or no Python headers to compile it against: the library itself
    needs neither, and the binding then marshals in Python."""
    import sysconfig
    if os.path.exists(HOST):
        os.remove(HOST)
    python_include = sysconfig.get_paths()["include"]
    try:
        import torch
        missing = None if os.path.exists(os.path.join(python_include, "Python.h")) else "Python.h"
    except ImportError:
        missing = "torch"
    if missing:
        print("_host.so: left out, %s is not there" % missing, flush=True)
        return None
    where = os.path.dirname(torch.__file__)
    tmp = HOST + ".tmp%d" % os.getpid()
    cmd = [host_compiler(), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(where, "include"),
           "-I", os.path.join(where, "include", "torch", "csrc", "api", "include"),
           "-I", python_include, "-o", tmp, os.path.join(CSRC, "host.cpp"),
           "-L", HERE, "-l:libmdsd.so", "-L", os.path.join(where, "lib"),
           "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, HOST)
    return HOST


def build(verbose: bool = True, extra=()) -> str:
    tag = ".tmp%d" % os.getpid()
    shutil.rmtree(OBJ, ignore_errors=True)
    os.makedirs(OBJ)

    def compile_one(src: str) -> str:
        obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
        cmd = [HIPCC, *FLAGS, *extra, "-c", "-o", obj, src]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        return obj

    with ThreadPoolExecutor(max_workers=jobs()) as pool:
        objs = list(pool.map(compile_one, sources()))
    tmp = LIB + tag
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    shutil.rmtree(OBJ, ignore_errors=True)
    build_host(verbose)
    return LIB


if __name__ == "__main__":
    build(extra=sys.argv[1:])
