"""Compile the HIP/C++ sources under csrc/ into libedgepipe.so (gfx950 only).

hipcc cross-compiles without a GPU.  Objects go to paper_2110_14895_amd/_build/
(ignored by git); the shared library is written next to this file so that it
travels with the source tree.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
OBJ_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libedgepipe.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
COMMON = ["-O3", "-std=c++17", "-fPIC", "-I", INCLUDE, "-I", CSRC, "-Wall", "-Wno-unused-function"]
# Kernel arguments arrive in scalar registers as far as those reach (14 words), instead of by a load from memory with which every launch would
# begin.  In LayerNorm, attention and the dense kernels of up to 256 x 256 tiles (bf16: streaming, one-tile, rows; fp32: direct, tile, rows) what is
# needed first therefore comes first in the arguments, and grid and block sizes, which are not among them, are arguments or constants; the persistent
# dense kernel and the embedding keep the order they had and read them.  The flag alone, builds in turn on one box: a layer of ViT-Large on 1 image
# 40.0 -> 38.1 us (seven launches), on 5 62.0 -> 60.2, of DeiT-Small on 1 28.2 -> 26.4, on 32 57.5 -> 56.0, of DeiT-Tiny on 64 52.6 -> 51.5.  Then the
# order, on another box: 38.0 -> 36.7, 62.3 -> 61.5, 26.5 -> 25.4, 59.0 -> 57.5, 52.0 -> 51.4.
HIP_FLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-mllvm", "-amdgpu-kernarg-preload-count=16"]
# Per-file additions.  The attention kernel takes maxima of matrix-pipe results; without the
# promise that the compiler need not quiet signalling NaNs it doubles every one of them with a
# canonicalising v_max (the hardware maxima and everything else stay IEEE: a NaN score still ends in NaN).
FILE_FLAGS = {"ep_attn_bf16.hip": ["-fno-honor-nans"]}


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, src.rsplit(".", 1)[0] + ".o")
    cmd = [HIPCC] + COMMON + HIP_FLAGS + FILE_FLAGS.get(src, []) + ["-c", os.path.join(CSRC, src), "-o", obj]
    if src.endswith(".cpp"):
        cmd.insert(1, "-x")
        cmd.insert(2, "hip")
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile of {src} failed:\n{r.stderr}")
    return obj


def build(jobs: int = 8) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        objs = list(pool.map(_compile, sources()))
    cmd = [HIPCC, "-shared", "-fPIC", "-Wl,-z,defs"] + HIP_FLAGS + ["-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    return LIB


if __name__ == "__main__":
    print(build())
    sys.exit(0)
