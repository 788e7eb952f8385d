"""Compile the HIP sources in csrc/ into paper_2509_09679_amd/libbq.so for gfx950 and the binding's caller, csrc/bqcall.c, into
the module bqcall of the Python that runs this (in-tree)."""
from __future__ import annotations

import glob
import importlib.machinery
import os
import shutil
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libbq.so")
CALL = os.path.join(HERE, "bqcall" + importlib.machinery.EXTENSION_SUFFIXES[0])

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# Packed-fp32 VALU instructions are switched off for every device translation unit.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Wno-unknown-attributes",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _compile(src: str, extra=()) -> str:
    obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
    cmd = [HIPCC, "-c", src, "-o", obj] + FLAGS + list(extra)
    subprocess.run(cmd, check=True)
    return obj


def build_caller() -> bool:
    """The binding calls through ctypes without it, so a machine that has no Python headers or no C compiler does without."""
    include = sysconfig.get_paths()["include"]
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None or not os.path.exists(os.path.join(include, "Python.h")):
        print("bqcall is not built (no C compiler or no Python.h): the binding's calls go through ctypes")
        if os.path.exists(CALL):
            os.remove(CALL)
        return False
    subprocess.run([cc, "-O2", "-Wall", "-shared", "-fPIC", "-I" + include, "-I" + os.path.join(ROOT, "include"),
                    os.path.join(CSRC, "bqcall.c"), "-o", CALL], check=True)
    return True


def build(verbose: bool = False, save_temps: bool = False) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    extra = ["-save-temps=obj"] if save_temps else []
    srcs = sources()
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(lambda s: _compile(s, extra), srcs))
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs
    subprocess.run(cmd, check=True)
    build_caller()
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    import sys

    build(verbose=True, save_temps="--save-temps" in sys.argv)
