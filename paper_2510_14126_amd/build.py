"""Build the gfx950 HIP library ``libpaged_attn.so`` in-tree with hipcc.

Every source is compiled for gfx950 only, with packed-fp32 instruction
selection disabled, and linked into one shared library next to this file;
``_pycall``, the CPython extension through which the binding makes its
per-step calls faster, is built beside it where a host compiler and Python's
headers are there.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "libpaged_attn.so")
SOURCES = ["api.cpp", "decode_mfma.hip", "cascade.hip", "reduce.hip", "append.hip", "extend.hip",
           "stream_copy.hip", "gather_tiles.hip", "noalloc.hip"]
PYCALL_PATH = os.path.join(HERE, "_pycall" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
ARCH = "gfx950"

COMMON_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
]


def hipcc() -> str:
    path = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(path):
        raise RuntimeError("hipcc not found; ROCm is required to build the library")
    return path


def host_compiler() -> str | None:
    path = shutil.which("g++") or "/opt/rocm/llvm/bin/clang++"
    return path if os.path.exists(path) else None


def build_pycall(verbose: bool = False) -> bool:
    """Build the extension; False (and none left behind) without a host
    compiler or Python's headers: the binding then calls through ctypes."""
    cc, include = host_compiler(), sysconfig.get_paths()["include"]
    if cc is None or not os.path.exists(os.path.join(include, "Python.h")):
        print("note: no host compiler or no Python.h: _pycall is not built, calls go through ctypes", file=sys.stderr)
        if os.path.exists(PYCALL_PATH):
            os.remove(PYCALL_PATH)
        return False
    tmp = PYCALL_PATH + ".tmp"
    _run([cc, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-fvisibility=hidden",
          "-I", include, "-I", os.path.join(HERE, "..", "include"),
          os.path.join(CSRC, "pycall.cpp"), "-o", tmp], verbose)
    os.replace(tmp, PYCALL_PATH)
    return True


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(line for line in (r.stdout + r.stderr).splitlines()
                    if "is not a recognized feature for this target" not in line)
    if r.returncode != 0:
        raise RuntimeError(f"command failed ({r.returncode}): {' '.join(cmd)}\n{out}")
    if verbose and out.strip():
        print(out)


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compile every source and link the shared library; returns its path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    cc = hipcc()
    include = ["-I", os.path.join(HERE, "..", "include"), "-I", CSRC]

    def compile_one(src):
        obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
        _run([cc, *COMMON_FLAGS, *include, "-c", os.path.join(CSRC, src), "-o", obj], verbose)
        return obj

    with ThreadPoolExecutor(min(jobs, len(SOURCES))) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = LIB_PATH + ".tmp"
    _run([cc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs], verbose)
    os.replace(tmp, LIB_PATH)
    build_pycall(verbose)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
