"""Compile libswz.so for gfx950 with hipcc, and the Python call path with the host compiler, in-tree (next to this file)."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libswz.so")
SOURCES = ["swz.hip"]
HEADERS = ["gemm_kernel.h", "gemm_subtile_kernel.h", "gemm_pair_kernel.h", "gemm_dispatch.h", "aux_kernels.h", "transpose_kernel.h", "transpose_dispatch.h", "tile_sweep.h", "rowwise_kernel.h", "row_dispatch.h", "mfma_peak_kernel.h", "pid_decode.h", os.path.join("..", "..", "include", "swz.h")]

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


FAST_DEPS = [FAST_SOURCE, os.path.join(HERE, "..", "include", "swz.h")]


def rocm_include() -> str:
    """Where hip/hip_runtime.h is: beside the hipcc that HIPCC names (a path, or a name to look up), or under ROCM_PATH or /opt/rocm."""
    hipcc = shutil.which(HIPCC)
    homes = [os.path.dirname(os.path.dirname(f)) for f in (hipcc, hipcc and os.path.realpath(hipcc)) if f]
    for home in homes + [os.environ.get("ROCM_PATH") or "/opt/rocm", "/opt/rocm"]:
        if os.path.exists(os.path.join(home, "include", "hip", "hip_runtime.h")):
            break
    return os.path.join(home, "include")


def fast_tag(torch) -> str:
    """What a _fastcall.so carries that was built for this torch."""
    return "swz built for torch " + torch.__version__


def fastcall_is_current(torch) -> bool:
    if not os.path.exists(FAST) or any(os.path.getmtime(FAST) < os.path.getmtime(d) for d in FAST_DEPS):
        return False
    with open(FAST, "rb") as f:
        return fast_tag(torch).encode() + b"\0" in f.read()


def build_fastcall(force: bool = True, verbose: bool = False) -> str | None:
    """_fastcall.so, against the torch of this interpreter.  Without one for ROCm there is none, and where it does not build there is none
    either, and a warning: every call works without it, 2 us slower."""
    try:
        import torch
    except ImportError:
        return None
    if torch.version.hip is None:
        return None
    if not force and fastcall_is_current(torch):
        return FAST
    base = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wno-attributes", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DSWZ_TORCH_TAG="{fast_tag(torch)}"', f"-I{base}/include",
           f"-I{base}/include/torch/csrc/api/include", f"-I{rocm_include()}", f"-I{sysconfig.get_paths()['include']}", FAST_SOURCE, "-o", FAST,
           f"-L{base}/lib", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        res = subprocess.run(cmd, capture_output=True, text=True)
        failed = f"{cmd[0]} failed ({res.returncode}):\n{res.stderr}" if res.returncode != 0 else None
    except OSError as e:
        failed = f"{cmd[0]}: {e}"
    if failed is not None:
        if os.path.exists(FAST):                    # of other sources or another torch
            os.remove(FAST)
        warnings.warn("_fastcall.so is not built, calls take the slower general path. " + failed, RuntimeWarning, stacklevel=2)
        return None
    return FAST


def build(force: bool = True, extra_flags: list[str] | None = None, verbose: bool = False) -> str:
    lib = build_lib(force, extra_flags, verbose)
    build_fastcall(force, verbose)
    return lib


def build_lib(force: bool = True, extra_flags: list[str] | None = None, verbose: bool = False) -> str:
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
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
