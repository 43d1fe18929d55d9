"""Compile the HIP sources into ``libprism.so`` (gfx950 only) and the marshalling of Python calls into the extension module
``_marshal``, both next to this file."""
import glob
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libprism.so")
# Named for the interpreter it is compiled for: another one does not find it and takes the general route of the binding.
MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))

# Packed-fp32 instructions are switched off for every HIP translation unit.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def hipcc_path():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def sources():
    return sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))


def build_marshal():
    """The Python extension module of ``csrc/marshal.cpp`` (host code; it is handed the library's addresses at run time).

    It only shortens ordinary calls, so where Python's headers or a host compiler are missing there is none (None is
    returned); raises on any compiler error."""
    include = sysconfig.get_paths()["include"]
    cxx = os.environ.get("CXX") or shutil.which("g++") or shutil.which("amdclang++") or shutil.which("c++")
    if not cxx or not os.path.exists(os.path.join(include, "Python.h")):
        print("no host compiler or no Python headers: calls from Python take the general route", file=sys.stderr)
        return None
    cmd = [cxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-I", include, os.path.join(HERE, "csrc", "marshal.cpp"),
           "-o", MARSHAL + ".tmp"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("compiling marshal.cpp failed:\n" + " ".join(cmd) + "\n" + res.stderr)
    os.replace(MARSHAL + ".tmp", MARSHAL)
    return MARSHAL


def build_library(verbose=False):
    """The C ABI and its kernels.  Always recompiles; raises on any compiler error."""
    cmd = [hipcc_path()] + [f for f in HIPCC_FLAGS if f] + [
        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc"),
    ] + sources() + ["-o", LIB + ".tmp"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + " ".join(cmd) + "\n" + err)
    if verbose and err.strip():
        print(err)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_marshal() or "")
