"""Build liblt.so (host C++ + HIP kernels for gfx950) in-tree.

Usage: python -m paper_2102_13267_amd.build [--force]
Every translation unit is compiled in parallel; objects live in paper_2102_13267_amd/_build/.
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "liblt.so")
REC = os.path.join(HERE, "_ltrec" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))   # recording fast path of the binding
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

HIP_SOURCES = ["lt_k_ew.hip", "lt_k_reduce.hip", "lt_k_rowop.hip", "lt_gemm.hip", "lt_gemm_bf16.hip", "lt_attention.hip", "lt_static_scratch.hip"]
CPP_SOURCES = ["lt_api.cpp", "lt_barrier.cpp", "lt_lower.cpp", "lt_schedule.cpp"]

# packed-fp32 VALU ops are switched off for all device code: some of their forms have given wrong
# results on this hardware, silently
HIP_FLAGS = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-value"]
CPP_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include"]


def _headers():
    return [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")] + \
           [os.path.join(HERE, "..", "include", "lt.h")]


def _stale(obj, src):
    if not os.path.exists(obj):
        return True
    t = os.path.getmtime(obj)
    return any(os.path.getmtime(p) > t for p in [src] + _headers())


def _compile(src, force):
    obj = os.path.join(OUT, os.path.basename(src) + ".o")
    if not force and not _stale(obj, src):
        return obj, ""
    if src.endswith(".hip"):
        cmd = [os.path.join(ROCM, "bin", "hipcc")] + HIP_FLAGS + ["-c", src, "-o", obj]
    else:
        cmd = ["g++"] + CPP_FLAGS + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    log = "\n".join(l for l in (r.stdout + r.stderr).splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{log}")
    return obj, log


def build(force: bool = False, verbose: bool = True) -> str:
    os.makedirs(OUT, exist_ok=True)
    srcs = [os.path.join(CSRC, s) for s in HIP_SOURCES + CPP_SOURCES]
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        results = list(ex.map(lambda s: _compile(s, force), srcs))
    objs = [o for o, _ in results]
    for _, log in results:
        if log.strip() and verbose:
            print(log)
    if force or not os.path.exists(LIB) or any(os.path.getmtime(o) > os.path.getmtime(LIB) for o in objs):
        cmd = [os.path.join(ROCM, "bin", "hipcc"), "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}{r.stderr}")
    # the binding's recording fast path: a CPython extension, plain C, no dependency on liblt.so
    rec_src = os.path.join(CSRC, "ltrec_module.c")
    if force or not os.path.exists(REC) or os.path.getmtime(rec_src) > os.path.getmtime(REC):
        cmd = ["gcc", "-O2", "-fPIC", "-shared", "-Wall", f"-I{sysconfig.get_paths()['include']}", rec_src, "-o", REC]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}{r.stderr}")
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
