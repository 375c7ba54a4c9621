"""Build the HIP shared library (gfx950) in-tree.

hipcc cross-compiles for gfx950 on a machine without a GPU. Flags:
  -ffp-contract=off   every FMA in the kernels is explicit, so identical
                      expressions round identically wherever they appear;
  -Xclang -target-feature -Xclang -packed-fp32-ops
                      no packed FP32 instructions are generated;
  -falign-loops=64    loops start at an instruction cache line: the traversal
                      loop takes up to 2 % longer where it does not (2^24 hair
                      pairs 1842 against 1812 us after a change before it).
"""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SRC = os.path.join(PKG, "csrc", "fiberhit.hip")
SRCS = [SRC, os.path.join(PKG, "csrc", "presplit.hip")]
OUT_DIR = os.path.join(PKG, "_lib")
LIB = os.path.join(OUT_DIR, "libfiberhit.so")
# the same sources with limits that large calls alone would meet set small, for
# the tests of what happens there: nodes a wave of pre-subdivision stacks,
# candidates of a list that one launch tests
LIB_SMALL = os.path.join(OUT_DIR, "libfiberhit_small_limits.so")
SMALL_LIMITS = ("-DFIBERHIT_NODE_STACK=64", "-DFIBERHIT_MAX_ROUNDS=3")
ARCH = "gfx950"


def hipcc_cmd(out: str, extra=()):
    return ["hipcc", f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-shared",
            "-ffp-contract=off", "-falign-loops=64",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-function",
            "-I", os.path.join(ROOT, "include"), *extra, "-o", out, *SRCS]


def build(verbose: bool = False, lib: str = LIB, extra=()) -> str:
    os.makedirs(OUT_DIR, exist_ok=True)
    tmp = lib + ".tmp"
    cmd = hipcc_cmd(tmp, extra)
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed")
    os.replace(tmp, lib)
    return lib


def build_small(verbose: bool = False) -> str:
    return build(verbose, LIB_SMALL, SMALL_LIMITS)


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
