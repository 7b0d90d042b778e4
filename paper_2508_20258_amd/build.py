"""Compile libswz.so for gfx950 with hipcc, and the Python call path with the host compiler, in-tree (next to this file)."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libswz.so")
SOURCES = ["swz.hip"]
HEADERS = ["gemm_kernel.h", "gemm_subtile_kernel.h", "gemm_dispatch.h", "aux_kernels.h", "transpose_kernel.h", "rowwise_kernel.h", "mfma_peak_kernel.h", "pid_decode.h", os.path.join("..", "..", "include", "swz.h")]

FAST_SOURCE = os.path.join(CSRC, "fastcall.cpp")
FAST = os.path.join(HERE, "_fastcall.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-shared", "-fPIC",
    # The library does not name a HIP runtime of its own: its hip* symbols bind to the runtime
    # the host process already uses (torch ships one), so kernels, streams and events all live in
    # one runtime.  A C program that links libswz links libamdhip64 itself.
    "-no-hip-rt",
    # packed-fp32 instructions are kept out of every kernel of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def build_fastcall(force: bool = True, verbose: bool = False) -> str | None:
    """_fastcall.so, against the torch of this interpreter; None without one (the host entry points work without it)."""
    try:
        import torch
    except ImportError:
        return None
    import sysconfig
    if not force and os.path.exists(FAST) and os.path.getmtime(FAST) >= os.path.getmtime(FAST_SOURCE):
        return FAST
    base = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(HIPCC))
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wno-attributes", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f"-I{base}/include", f"-I{base}/include/torch/csrc/api/include",
           f"-I{rocm}/include", f"-I{sysconfig.get_paths()['include']}", FAST_SOURCE, "-o", FAST, f"-L{base}/lib", "-lc10", "-lc10_hip", "-ltorch_cpu",
           "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed ({res.returncode}):\n{res.stderr}")
    return FAST


def build(force: bool = True, extra_flags: list[str] | None = None, verbose: bool = False) -> str:
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    build_fastcall(force, verbose)
    deps = srcs + [os.path.join(CSRC, h) for h in HEADERS]
    if not force and os.path.exists(LIB) and all(os.path.getmtime(LIB) >= os.path.getmtime(d) for d in deps):
        return LIB
    cmd = [HIPCC, *FLAGS, *(extra_flags or []), *srcs, "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "packed-fp32-ops"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{err}")
    if verbose and err.strip():
        print(err, file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
