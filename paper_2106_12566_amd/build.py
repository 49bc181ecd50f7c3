"""Compile the HIP sources of the package into ``libkrpe.so`` (gfx950).

    python -m paper_2106_12566_amd.build          # or: python paper_2106_12566_amd/build.py

The library is built in-tree, next to this file, so that it travels with the
source tree.  Packed-FP32 instruction selection is disabled for all device
code (``-packed-fp32-ops``).
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libkrpe.so")
SOURCES = [os.path.join(HERE, "csrc", f) for f in ("kernels.hip", "grad_bias.hip", "direct.hip", "bwd_direct.hip", "bwd_exact.hip", "toeplitz.hip", "phi.hip",
                                                   "long_seq.hip", "api.hip")]
# The convolution kernel at N = 16384, compiled on its own with LLVM's
# maximum-ILP machine scheduler (measured faster for that length only).
TOP = os.path.join(HERE, "csrc", "conv_top.hip")
TOP_FLAGS = ["-mllvm", "-amdgpu-sched-strategy=max-ilp"]
ARCH = "gfx950"


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the ROCm toolchain is required to build libkrpe.so")


def _flags() -> list[str]:
    return [
        f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-Wall", "-Wno-unused-function",
        "-I", os.path.join(ROOT, "include"),
    ]


def command(out: str = LIB) -> list[str]:
    """One hipcc run compiling and linking every source into `out`."""
    return [hipcc(), *_flags(), "-shared", "-o", out, TOP, *SOURCES]


def object_command(src: str, obj: str) -> list[str]:
    return [hipcc(), *_flags(), *(TOP_FLAGS if src == TOP else []), "-c", "-o", obj, src]


def link_command(objs: list[str], out: str) -> list[str]:
    return [hipcc(), f"--offload-arch={ARCH}", "-fPIC", "-shared", "-o", out, *objs]


def _run(cmd: list[str], verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{res.stdout}\n{res.stderr}")


def build(verbose: bool = False) -> str:
    """Compile libkrpe.so (always recompiles, the sources side by side); return its path."""
    tmp = LIB + ".tmp"
    sources = [TOP, *SOURCES]
    objs = [f"{LIB}.{os.path.splitext(os.path.basename(s))[0]}.o" for s in sources]
    try:
        with ThreadPoolExecutor(max_workers=min(len(sources), os.cpu_count() or 1)) as pool:
            list(pool.map(lambda so: _run(object_command(*so), verbose), zip(sources, objs)))
        _run(link_command(objs, tmp), verbose)
    finally:
        for o in objs:
            if os.path.exists(o):
                os.remove(o)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-q" not in sys.argv))
