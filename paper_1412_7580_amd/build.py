"""Build libfftconv.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libfftconv.so")
SOURCES = ["api.hip", "fft_kernels.hip", "fft_kernels_mixed_small.hip", "fft_kernels_mixed_large.hip", "fft1d_mixed.hip",
           "fft_kernels_natural.hip", "fft_rect_fwd.hip", "fft_rect_inv.hip", "fft_thin_inv.hip", "fused_small.hip", "cgemm_kernels.hip", "cgemm_bingroup.hip", "cgemm_thin.hip", "cgemm_direct.hip", "cgemm_split.hip"]
HEADERS = ["fft_core.hpp", "fft_kernels_impl.hpp", "fft_rect_impl.hpp", "kernels.hpp", "thin.hpp", "gemm_params.hpp", "gemm_rules.hpp", "bf16_split.hpp", os.path.join("..", "..", "include", "fftconv.h")]
FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(os.path.join(CSRC, s)) > t for s in SOURCES + HEADERS)


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every source to an object (in parallel) and link the shared library."""
    if not force and not stale():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(OBJ, src.replace(".hip", ".o"))
        cmd = [hipcc] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        return obj

    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
