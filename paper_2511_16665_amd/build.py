"""Builds libtlt.so (the HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

Run as `python -m paper_2511_16665_amd.build`.  Cross-compiles without a GPU.
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libtlt.so")
SOURCES = ["api.hip", "gemm.hip", "attn.hip", "elementwise.hip", "sample.hip", "mab.cpp", "ngram.cpp", "tmpl.cpp"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function",
         # a kernel's first 16 argument words arrive in scalar registers with the wave instead of being loaded by it: plain arguments that a
         # kernel needs first stand before its structs (plain decoding of one sequence 12.65 -> 12.50 ms a pass, 16 sequences 17.42 -> 17.21, 16 x 16 nodes 22.24 -> 22.03)
         "-mllvm", "-amdgpu-kernarg-preload-count=16",
         "-Wno-inline-asm"]   # (m0 is set inside the asm blocks that issue global->LDS loads: the clobber is intended)


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    # host-only sources (.cpp) need none of the device flags
    flags = FLAGS if src.endswith(".hip") else ["-O2", "-std=c++17", "-fPIC", "-Wall"]
    cmd = ["hipcc", *flags, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + f".tmp{os.getpid()}"
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp])
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
