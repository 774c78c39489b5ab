"""Build libsegsalsa.so (gfx950) in-tree with hipcc.

Usage: python -m paper_1504_07028_amd.build [-v]
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsegsalsa.so")
# (source, macros): the prox kernel's builds are compiled in parts, side by side
SOURCES = [*(("prox_kernel.hip", (f"SEGSALSA_PROX_BITS={bits}", f"SEGSALSA_PROX_PART={part}"))
             for bits in (64, 32) for part in (4, 0, 2)),
           ("adjoint_kernels.hip", ()), ("fft_kernels.hip", ()), ("api.hip", ()), ("fft_pow2_kernels.hip", ()),
           ("fft_blu_kernels.hip", ()), ("tri_kernels.hip", ()), ("win_kernels.hip", ()), ("misc_kernels.hip", ()),
           ("residual_kernels.hip", ())]
ARCH = "gfx950"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
COMMON = [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
          # no packed FP32 instructions in the device code
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-I", INCLUDE, "-I", CSRC]


def _compile(src: str, macros: tuple, verbose: bool) -> str:
    obj = os.path.join(BUILD_DIR, "-".join([os.path.splitext(src)[0], *macros]).replace("=", "") + ".o")
    cmd = [HIPCC, *COMMON, *(f"-D{m}" for m in macros), "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return obj


def build(verbose: bool = False) -> str:
    """Compile every HIP source for gfx950 and link libsegsalsa.so; returns its path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(lambda s: _compile(*s, verbose), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv[1:]))
