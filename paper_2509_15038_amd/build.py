"""Compile the HIP sources into paper_2509_15038_amd/libcurdkv.so for gfx950, and the CPython module
_call beside it (argument marshalling, no device code; its file name ends as this interpreter's modules do).

    python -m paper_2509_15038_amd.build

hipcc cross-compiles without a GPU.  Nothing is built lazily at import time:
tests, the smoke check and the benchmark load the library this step left here.
"""

from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libcurdkv.so")
CALL = os.path.join(HERE, "_call" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
SOURCES = ["curdkv_api.hip", "scores_kernels.hip", "select_kernels.hip", "split_select.hip", "compact_kernels.hip", "fused_kernel.hip", "adaptive_kernels.hip",
           "sketch_host.cpp"]


def _build_call_module(hipcc: str, verbose: bool) -> None:
    """The CPython module.  Where there is no Python.h or no C++ compiler the binding does without it."""
    headers = sysconfig.get_paths()["include"]
    compilers = [os.environ.get("CXX"), "g++", "clang++", os.path.join(os.path.dirname(hipcc), "amdclang++")]
    cxx = next((path for path in map(shutil.which, filter(None, compilers)) if path), None)
    if not cxx or not os.path.exists(os.path.join(headers, "Python.h")):
        if os.path.exists(CALL):                    # (of an older source)
            os.remove(CALL)
        print("no Python.h or no C++ compiler: the binding marshals its arguments through ctypes (1 us a call slower)", flush=True)
        return
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", headers, "-I", os.path.join(ROOT, "include"),
           os.path.join(HERE, "csrc", "call_module.cpp"), "-o", CALL]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)


def build(verbose: bool = True) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
           "-fno-gpu-rdc", "-Wall", "-Wno-unused-function",
           # packed fp32 VALU forms are switched off for all device code
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc")]
    cmd += ["-x", "hip"] + [os.path.join(HERE, "csrc", s) for s in SOURCES]
    cmd += ["-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    _build_call_module(hipcc, verbose)
    return LIB


if __name__ == "__main__":
    build()
    print("built", LIB)
    sys.exit(0)
