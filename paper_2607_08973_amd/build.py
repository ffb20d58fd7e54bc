"""Build libsifar.so in-tree with hipcc for gfx950 (MI355X).

Usage: ``python -m paper_2607_08973_amd.build`` (or ``build()`` from Python).
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libsifar.so")
SOURCES = [os.path.join(CSRC, "kernels.hip"), os.path.join(CSRC, "floors.hip"),
           os.path.join(CSRC, "litmus.hip"), os.path.join(CSRC, "noalloc.hip"),
           os.path.join(CSRC, "api.cpp")]
ARCH = "gfx950"

FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-ffp-contract=off",
    # no packed fp32 instructions (v_pk_add_f32 and friends) in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # leading scalar kernel arguments preloaded into SGPRs at wave start
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall",
    "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: ROCm is required to build libsifar")


def build(verbose: bool = False, lib: str = LIB, defines: tuple = ()) -> str:
    """Compile every HIP/C++ source into libsifar.so (always recompiles), or
    into `lib` with preprocessor `defines`."""
    tmp = lib + ".tmp"
    cmd = [hipcc(), *FLAGS, *[f"-D{d}" for d in defines], "-I", INCLUDE, "-I", CSRC, *SOURCES,
           "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(l for l in (res.stdout + res.stderr).splitlines()
                    if "packed-fp32-ops" not in l and "warning generated" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{out}")
    if verbose and out.strip():
        print(out, file=sys.stderr)
    os.replace(tmp, lib)
    return lib


if __name__ == "__main__":
    print(build(verbose=True))
