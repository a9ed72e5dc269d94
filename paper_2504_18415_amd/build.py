"""Builds libhbitlinear.so (HIP, gfx950 only) in-tree with hipcc, and with g++ the binding's native half, _host_call.so.

Usage: ``python -m paper_2504_18415_amd.build [--incremental]`` or ``build.build_library()``.
The sources are cross-compiled, so no GPU is needed to build.  Every translation unit is compiled by a
process of its own (in parallel) into ``csrc/_build/`` and the objects are linked into the library;
``incremental=True`` recompiles only the units older than their source or than any header.
"""
from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ_DIR = os.path.join(CSRC, "_build")
LIB = os.path.join(PKG, "libhbitlinear.so")
HOST_CALL = os.path.join(PKG, "_host_call.so")
SOURCES = ["api.hip", "fwht_quant.hip", "ternary_setup.hip", "ternary_gemm.hip", "ternary_gemm_f6f4.hip", "mid_gemm.hip",
           "decode_gemm.hip", "fused_small.hip", "fused_bytes.hip", "kv_quant.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off",                       # butterflies and scales round once per operation
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument", "-Wno-inline-asm",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass warns that it does not know the packed-fp32 target feature: harmless
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        sys.stderr.write(err + "\n")
        raise RuntimeError("compilation failed: " + " ".join(cmd[-3:]))
    if verbose and err.strip():
        print(err)


def _host_call_command(out):
    """host_call.cpp is host code against torch's own headers and libraries (the ones that hbl.py imports)."""
    import sysconfig

    import torch
    base = os.path.dirname(torch.__file__)
    include = os.path.join(base, "include")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            "-isystem", include, "-isystem", os.path.join(include, "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
            "-isystem", sysconfig.get_paths()["include"], "-I" + os.path.join(ROOT, "include"),
            os.path.join(CSRC, "host_call.cpp"), "-o", out,
            "-L" + os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]


def build_library(verbose: bool = False, extra_flags=(), incremental: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ_DIR, exist_ok=True)
    headers = glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    newest_header = max(os.path.getmtime(h) for h in headers)
    jobs, objs = [], []
    for s in SOURCES:
        src = os.path.join(CSRC, s)
        obj = os.path.join(OBJ_DIR, s.replace(".hip", ".o"))
        objs.append(obj)
        fresh = (incremental and not extra_flags and os.path.exists(obj)
                 and os.path.getmtime(obj) > max(os.path.getmtime(src), newest_header))
        if not fresh:
            jobs.append([hipcc, *HIPCC_FLAGS, *extra_flags, "-c", src, "-o", obj])
    host_src, host_tmp = os.path.join(CSRC, "host_call.cpp"), HOST_CALL + f".tmp{os.getpid()}"
    host_stale = not (incremental and os.path.exists(HOST_CALL)
                      and os.path.getmtime(HOST_CALL) > max(os.path.getmtime(host_src), newest_header))
    if host_stale:
        jobs.append(_host_call_command(host_tmp))
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, max(len(jobs), 1))) as pool:
        for f in [pool.submit(_run, cmd, verbose) for cmd in jobs]:
            f.result()
    tmp = LIB + f".tmp{os.getpid()}"
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp], verbose)
    os.replace(tmp, LIB)
    if host_stale:
        os.replace(host_tmp, HOST_CALL)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True, incremental="--incremental" in sys.argv))
