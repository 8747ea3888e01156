"""Compile libsdpm.so (all HIP sources, gfx950) in place, next to this file.

Usage:  python -m paper_1709_04703_amd.build   (or build() from Python)
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsdpm.so")
SOURCES = ["capi.hip", "mesh.hip", "tile.hip", "ade.hip", "fft.hip", "pk.hip", "particles.hip", "sort.hip", "net.hip", "cosmology.cpp", "profiler.cpp"]
ARCH = os.environ.get("SDPM_OFFLOAD_ARCH", "gfx950")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared", f"--offload-arch={ARCH}",
    # packed FP32 instructions are disabled for every HIP translation unit
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]
LIBS = ["-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib"]


def hipcc() -> str:
    path = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(path):
        raise RuntimeError("hipcc not found")
    return path


def build(verbose: bool = False) -> str:
    srcs = []
    for s in SOURCES:
        p = os.path.join(CSRC, s)
        srcs += ["-x", "hip", p]
    tmp = LIB + ".tmp"
    cmd = [hipcc()] + FLAGS + srcs + LIBS + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("libsdpm build failed")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
