"""Build liblasad.so (hand-written HIP, gfx950 only) in-tree with hipcc, and _steps.so, the marshalling of the calls
(host code against torch's C++ interface), with g++.

Usage: ``python -m paper_2507_01652_amd.build``.  Both land next to this
file so that they travel with the source tree; nothing is JIT-compiled at import.
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "liblasad.so")
STEPS = os.path.join(_HERE, "_steps.so")

SOURCES = [
    "lasad_api.hip",
    "lasad_decay.hip",
    "lasad_forward_generic.hip",
    "lasad_forward_scan.hip",
    "lasad_forward_f32_chunk.hip",
    "lasad_forward_mfma.hip",
    "lasad_forward_mfma_ws.hip",
    "lasad_forward_scalar_chunk.hip",
    "lasad_forward_gated_chunk.hip",
    "lasad_decode.hip",
    "lasad_decode_cached.hip",
    "lasad_backward.hip",
    "lasad_backward_gated.hip",
    "lasad_backward_gated_mfma.hip",
    "lasad_backward_gated_chunk.hip",
    "lasad_backward_layer.hip",
]

# Packed-fp32 instruction selection is switched off for every HIP translation unit.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def build_steps(verbose: bool = False) -> str:
    """Compile the CPython extension and link it to the liblasad.so beside it."""
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-w",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__=1",
           "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(rocm, "include")]
    for path in cpp_extension.include_paths():
        cmd += ["-isystem", path]
    cmd += [os.path.join(CSRC, "lasad_steps.cpp"), "-o", STEPS, LIB, "-Wl,-rpath,$ORIGIN"]
    for path in cpp_extension.library_paths():
        cmd += ["-L" + path]
    cmd += ["-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return STEPS


def build(verbose: bool = False, extra_flags=(), jobs: int | None = None) -> str:
    """Compile every source to an object (several at a time) in a temporary folder, then link the library."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    jobs = jobs or max(1, min(8, os.cpu_count() or 1))
    with tempfile.TemporaryDirectory(prefix="lasad_build_") as tmp:
        def compile_one(src):
            obj = os.path.join(tmp, src + ".o")
            cmd = [hipcc, *FLAGS, *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj
        with ThreadPoolExecutor(max_workers=jobs) as pool:
            objs = list(pool.map(compile_one, SOURCES))
        cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-soname,liblasad.so", *objs, "-o", LIB]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
    build_steps(verbose)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra_flags=sys.argv[1:])
    print("built", LIB)
