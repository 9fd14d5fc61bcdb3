"""Compile the HIP sources into paper_2602_12271_amd/libmonarchrt.so for gfx950.

    python -m paper_2602_12271_amd.build

hipcc cross-compiles without a GPU.  The library is built in-tree so that it travels
with the source tree to the machine that runs it.
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
SOURCES = ["mrt_api.cpp", "mrt_static.hip", "mrt_f32.hip", "mrt_f32_bf16io.hip", "mrt_bf16.hip", "mrt_dense_bf16.hip", "mrt_bwd_f32.hip", "mrt_bwd_bf16.hip",
           "mrt_bwd_waves_bf16.hip"]
OUT = os.path.join(HERE, "libmonarchrt.so")

FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-shared",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
    # packed fp32 instructions are kept out of the generated code on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # max / min / select need no NaN-quieting instructions: a NaN in the inputs gives an
    # unspecified result either way; infinities are honoured (the masks are -inf)
    "-fno-honor-nans",
    "-Wno-unused-command-line-argument",
]


# Kernels of more than 256 registers: matrix results go to the registers that other instructions can name
# and only accumulators that live across steps to the rest (the default writes all of them to the rest and
# moves them back: 154 of 616 moves less in a 3000-instruction step, 1 to 4 % of the calls).
SOURCE_FLAGS = {"mrt_bwd_waves_bf16.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}


def build(verbose: bool = True) -> str:
    """Compiles every source to an object file (in parallel, under the git-ignored _build/) and
    links them into the library next to this file."""
    from concurrent.futures import ThreadPoolExecutor

    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    compile_flags = [f for f in FLAGS if f != "-shared"]

    def compile_one(src: str) -> str:
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        cmd = ["hipcc"] + compile_flags + SOURCE_FLAGS.get(src, []) + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines()
                        if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
        if r.returncode != 0:
            sys.stderr.write(r.stdout + r.stderr)
            raise RuntimeError("hipcc failed on " + src)
        if verbose and err.strip():
            print(err)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as pool:
        objs = list(pool.map(compile_one, SOURCES))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", OUT + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("link failed")
    os.replace(OUT + ".tmp", OUT)
    return OUT


if __name__ == "__main__":
    build()
