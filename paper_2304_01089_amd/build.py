"""Builds librptq.so (gfx950) in-tree with hipcc.  `python -m paper_2304_01089_amd.build`."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor
from typing import Optional

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "librptq.so")
# the binding's native argument marshalling (csrc/calls.cpp); the suffix keeps other interpreters from loading it
CALLS = os.path.join(PKG, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["host.cpp", "api.cpp", "calib_minmax.hip", "fold.hip", "ln_quant.hip", "ln_rows.hip", "gemm.hip", "gemm_small.hip", "kv_cache.hip", "ln_scatter.hip", "method1.hip"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-ffp-contract=off",
    # packed fp32 ALU forms are kept out of the generated code on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def _compile(src: str, objdir: str, verbose: bool) -> str:
    obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
    extra = os.environ.get("RPTQ_EXTRA_FLAGS", "").split()
    cmd = [hipcc(), "-x", "hip", *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, res.stdout, res.stderr))
    if verbose and res.stderr.strip():
        lines = [l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l]
        if lines:
            sys.stderr.write("\n".join(lines) + "\n")
    return obj


def build_calls() -> Optional[str]:
    """Compile the CPython module beside the library (host code only).  Where there is no C++ compiler of the host's, or no
    header of this Python's, there is no module (None): the binding does the same in Python."""
    untagged = os.path.join(os.path.dirname(CALLS), "_calls.so")
    if os.path.exists(untagged):                 # (any interpreter would load it)
        os.remove(untagged)
    include = sysconfig.get_paths()["include"]
    lacks = [what for what, there in (("g++", shutil.which("g++")), ("Python.h", os.path.exists(os.path.join(include, "Python.h"))))
             if not there]
    if lacks:
        sys.stderr.write("no native marshalling of calls: %s not found\n" % " and ".join(lacks))
        if os.path.exists(CALLS):                # (of an older source)
            os.remove(CALLS)
        return None
    tmp = CALLS + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", os.path.join(ROOT, "include"),
           "-I", include, os.path.join(CSRC, "calls.cpp"), "-o", tmp]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed for calls.cpp:\n%s\n%s" % (res.stdout, res.stderr))
    os.replace(tmp, CALLS)
    return CALLS


def build_library(verbose: bool = False, jobs: int = 6) -> str:
    """Compile every source for gfx950 and link the shared library; returns its path."""
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        objs = list(pool.map(lambda s: _compile(s, objdir, verbose), SOURCES))
    lib = os.environ.get("RPTQ_LIBRARY_OUT", LIB)
    tmp = lib + ".tmp"
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (res.stdout, res.stderr))
    os.replace(tmp, lib)
    build_calls()
    return lib


if __name__ == "__main__":
    print(build_library(verbose=True))
