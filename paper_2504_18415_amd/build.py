"""Builds libhbitlinear.so (HIP, gfx950 only) in-tree with hipcc, and with g++ the binding's native half, the extension module
_host_call.  The library needs neither g++ nor torch's headers: where the module cannot be built the binding goes without it.

Usage: ``python -m paper_2504_18415_amd.build [--incremental]`` or ``build.build_library()``.
The sources are cross-compiled, so no GPU is needed to build.  Every translation unit is compiled by a
process of its own (in parallel) into ``csrc/_build/`` and the objects are linked into the library;
``incremental=True`` recompiles only the units older than their source or than any header (the module also for another torch,
Python or command).
"""
from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ_DIR = os.path.join(CSRC, "_build")
LIB = os.path.join(PKG, "libhbitlinear.so")
HOST_CALL = os.path.join(PKG, "_host_call" + sysconfig.get_config_var("EXT_SUFFIX"))   # (its name says for which Python)
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
    import torch
    base = os.path.dirname(torch.__file__)
    include = os.path.join(base, "include")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DHBL_BUILT_FOR="{torch.__version__}"',
            "-isystem", include, "-isystem", os.path.join(include, "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
            "-isystem", sysconfig.get_paths()["include"], "-I" + os.path.join(ROOT, "include"),
            os.path.join(CSRC, "host_call.cpp"), "-o", out,
            "-L" + os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]


def _build_host_call(verbose, incremental, newest_header):
    """Compiles the module, or leaves none: one of another build must not be taken for this one's."""
    src, tmp, stamp = os.path.join(CSRC, "host_call.cpp"), HOST_CALL + f".tmp{os.getpid()}", os.path.join(OBJ_DIR, "host_call.stamp")
    untagged = os.path.join(PKG, "_host_call.so")
    if os.path.exists(untagged):
        os.remove(untagged)
    try:
        cmd = _host_call_command(tmp)
        made_by = sys.version + "\n" + "\n".join(cmd).replace(tmp, HOST_CALL)
        if (incremental and os.path.exists(HOST_CALL) and os.path.exists(stamp) and open(stamp).read() == made_by
                and os.path.getmtime(HOST_CALL) > max(os.path.getmtime(src), newest_header)):
            return
        _run(cmd, verbose)
        os.replace(tmp, HOST_CALL)
        with open(stamp, "w") as f:
            f.write(made_by)
    except Exception as e:   # no torch, no headers, no compiler, or they do not agree
        for path in (HOST_CALL, tmp):
            if os.path.exists(path):
                os.remove(path)
        sys.stderr.write(f"host_call.cpp was not built, hbl.py goes without it: {e}\n")


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
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(jobs) + 1)) as pool:
        host = pool.submit(_build_host_call, verbose, incremental, newest_header)
        for f in [pool.submit(_run, cmd, verbose) for cmd in jobs]:
            f.result()
        host.result()
    tmp = LIB + f".tmp{os.getpid()}"
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True, incremental="--incremental" in sys.argv))
