"""Build of the HIP library libmcrt.so for gfx950 (in-tree)."""
from __future__ import annotations

import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmcrt.so")
SOURCES = ["kernels.hip", "prep.hip", "transport.hip", "flight.hip", "slab.hip", "chords.hip", "api.cpp"]

# -ffp-contract=off keeps every FP64 expression in the order it is written
# (no fused multiply-add), so the FP64 path agrees with an independent FP64
# evaluation to the last bits of the math library.  Packed FP32 instructions
# are disabled for all device code.
HIPFLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-function", "-I" + os.path.join(ROOT, "include")]


# The transport kernels' loops hold rare code (sampling, births, phase
# functions) whose many FP64 constants the machine-level loop-invariant motion
# would keep in registers throughout: of the one-kernel transport 127 VGPRs and
# 4 spilled in place of 101 in the mixed form, 128 and 34 spilled in place of 119
# in the FP64 form; of the flights 128 and 3 in place of 107, 128 and 14 in place
# of 125.
SOURCE_FLAGS = {s: ["-mllvm", "-disable-machine-licm"] for s in ("transport.hip", "flight.hip")}


def hipcc() -> str:
    return shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def build_library(verbose: bool = False) -> str:
    objs = []
    build_dir = os.path.join(HERE, "_build")
    os.makedirs(build_dir, exist_ok=True)
    for src in SOURCES:
        obj = os.path.join(build_dir, src + ".o")
        lang = ["-x", "hip"] if src.endswith(".hip") else ["-x", "hip"]
        cmd = [hipcc()] + HIPFLAGS + SOURCE_FLAGS.get(src, []) + lang + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        objs.append(obj)
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
