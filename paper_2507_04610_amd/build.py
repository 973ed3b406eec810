"""Compile libany4.so (HIP, gfx950) in-tree with hipcc, and with g++ the torch extension that calls it.  `python -m paper_2507_04610_amd.build`."""
from __future__ import annotations

import glob
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libany4.so")
TORCH_SRC = os.path.join(CSRC, "any4_torch.cpp")
TORCH_EXT = os.path.join(PKG, "_any4_torch.so")
BENCH_SRC = os.path.join(PKG, "bench_support", "stream_read.hip")
BENCH_LIB = os.path.join(PKG, "bench_support", "libany4_bench.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-fno-gpu-flush-denormals-to-zero",            # sub-normal table entries dequantise as IEEE says
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-attributes",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def torch_extension_command():
    """host code only (no kernels): torch's headers and libraries, linked to libany4.so next to it"""
    import sysconfig
    from torch.utils import cpp_extension
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    includes = [os.path.join(ROOT, "include"), *cpp_extension.include_paths(), os.path.join(rocm, "include"),
                sysconfig.get_paths()["include"]]
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-w",
            *[f"-I{d}" for d in includes], TORCH_SRC, "-o", TORCH_EXT,
            *[f"-L{d}" for d in cpp_extension.library_paths()], "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10",
            "-lc10_hip", f"-L{PKG}", "-lany4", "-Wl,-rpath,$ORIGIN"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build_library(verbose: bool = True) -> str:
    """Always recompiles every source (seconds per file) and links libany4.so."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = []
    procs = []
    for src in sources():
        obj = os.path.join(objdir, os.path.basename(src) + ".o")
        objs.append(obj)
        cmd = [hipcc, *HIPCC_FLAGS, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd)))
    for src, p in procs:
        if p.wait() != 0:
            raise RuntimeError(f"hipcc failed on {src}")
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    cmd = torch_extension_command()
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    # bench.py's measurement helper (a read-only kernel): a library of its own, not part of libany4
    cmd = [hipcc, *HIPCC_FLAGS, "-shared", BENCH_SRC, "-o", BENCH_LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    build_library()
    sys.exit(0)
