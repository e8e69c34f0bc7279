"""Build ``libmooncake_hip.so`` (hipcc for gfx950, cross-compiles without a GPU) and ``_mccall``, through which the binding
calls it, in-tree."""
from __future__ import annotations

import os
import platform
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libmooncake_hip.so")
# the name says which interpreter it is for: others do not load it
CALLER = os.path.join(PKG, "_mccall" + sysconfig.get_config_var("EXT_SUFFIX"))
# host_plan.cpp holds no device code: hipcc compiles it as plain C++
SOURCES = ["mc_api.hip", "host_plan.cpp", "attn_prefill.hip", "attn_prefill_bf16.hip", "attn_narrow.hip", "attn_noalloc.hip", "kv_copy.hip", "prefix_hash.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# packed-fp32 VALU forms are switched off on purpose (device code only)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines()
                    if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _build_caller() -> None:
    """Where it cannot be built (no headers of this Python, another processor) the binding calls through ctypes."""
    untagged = os.path.join(PKG, "_mccall.so")           # any Python would load it
    if os.path.exists(untagged):
        os.remove(untagged)
    include, cxx = sysconfig.get_paths()["include"], os.environ.get("CXX", "g++")
    if not os.path.exists(os.path.join(include, "Python.h")) or shutil.which(cxx) is None or platform.machine() != "x86_64":
        sys.stderr.write(f"no _mccall for this Python (needs x86-64, {cxx} and {include}/Python.h): calls go through ctypes\n")
        return
    subprocess.run([cxx, "-O2", "-std=c++17", "-fPIC", "-Wall", "-shared", "-I", include, "-o", CALLER,
                    os.path.join(CSRC, "pycall.cpp")], check=True)


def build(verbose: bool = False) -> str:
    """Compile every kernel source and link the shared library; returns its path."""
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        caller = ex.submit(_build_caller)
        objs = list(ex.map(_compile, SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    caller.result()
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
