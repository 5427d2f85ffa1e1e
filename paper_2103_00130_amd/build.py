"""Build libabftgemm.so (hand-written HIP, gfx950 only) in-tree with hipcc."""
from __future__ import annotations

import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libabftgemm.so")
FASTCALL = os.path.join(HERE, "_fastcall.so")
SOURCES = ["api.hip", "pack.hip", "gemm_tile.hip", "gemm_tile_a256.hip", "gemm_tile_a256w24.hip", "gemm_tile_a256w42.hip",
           "gemm_tile_a128.hip", "gemm_tile_a64.hip", "gemm_tile_a64r4.hip", "gemm_tile_a64s.hip", "gemm_tile_g64.hip", "gemm_smallm.hip",
           "gemm_tile_wk32x32w4.hip", "gemm_tile_wk32x32w8.hip", "gemm_tile_wk32x32w8s.hip", "gemm_tile_wk32x64w4.hip", "gemm_tile_wk32x64w8.hip", "gemm_tile_wk64x64w4.hip",
           "rowops.hip", "locate.hip", "eb.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", "-Wno-inline-asm",
    # packed-FP32 instruction selection is switched off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-ffp-contract=off",
]


def build_library(force: bool = True, verbose: bool = False, clock_trace: bool = False) -> str:
    """clock_trace: build libabftgemm_clocktrace.so instead, the same sources with ABFT_CLOCK_TRACE defined (tiled
    kernels record cycle and wall counters per workgroup; load it through ABFT_LIBRARY, see bench.py --clock-trace)."""
    if clock_trace:
        return _build(force, verbose, os.path.join(HERE, "_build_clocktrace"), os.path.join(HERE, "libabftgemm_clocktrace.so"),
                      ["-DABFT_CLOCK_TRACE"])
    return _build(force, verbose, os.path.join(HERE, "_build"), LIB, [])


def _build(force, verbose, build_dir, lib, extra) -> str:
    os.makedirs(build_dir, exist_ok=True)
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC)] + [os.path.join(HERE, "..", "include", h) for h in ("abft_gemm.h", "abft_eb.h")]
    newest = max(os.path.getmtime(d) for d in deps)
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(build_dir, src.replace(".hip", ".o"))
        objs.append(obj)
        if force or not os.path.exists(obj) or os.path.getmtime(obj) < newest:
            cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = False
    for src, pr in procs:
        out, _ = pr.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if pr.returncode != 0:
            failed = True
            print(f"---- {src} failed ----\n{out}", file=sys.stderr)
        elif verbose and out.strip():
            print(f"---- {src} ----\n{out}")
    if failed:
        raise RuntimeError("hipcc failed")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *objs], check=True)
    return lib


def build_fastcall(force: bool = True) -> str:
    """_fastcall.so: the native marshalling that binding.py uses for the two calls of a serving loop (host code only)."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    src = os.path.join(CSRC, "fastcall.cpp")
    deps = [src] + [os.path.join(HERE, "..", "include", h) for h in ("abft_gemm.h", "abft_eb.h")]
    if not force and os.path.exists(FASTCALL) and os.path.getmtime(FASTCALL) >= max(os.path.getmtime(d) for d in deps):
        return FASTCALL
    lib_dir = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *(f"-isystem{d}" for d in cpp_extension.include_paths()), f"-I{sysconfig.get_paths()['include']}",
           src, "-o", FASTCALL, f"-L{lib_dir}", "-ltorch_python", "-ltorch_cpu", "-lc10"]
    subprocess.run(cmd, check=True)
    return FASTCALL


if __name__ == "__main__":
    print(build_fastcall(force="--force" in sys.argv))
    print(build_library(force="--force" in sys.argv, verbose=True, clock_trace="--clock-trace" in sys.argv))
