"""Builds libhatmid.so (HIP, gfx950) in-tree.  `python -m paper_2503_18989_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhatmid.so")
SOURCES = ["api.hip", "gemm.hip", "attention.hip", "elementwise.hip", "peaks.hip", "sched.cpp"]   # sched.cpp: host code only
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 VALU forms
         "-Wno-unused-result"]
# The GEMM main loops start on a 128-byte boundary.  Left to chance, their place moves with every instruction of the code before
# them, and with it their time: 28.3 .. 30.9 us for the down product of 256 rows (7B shape) unaligned and at 32, 64, 128 and 256 bytes,
# 143 .. 145 us for gate/up of 512 rows (13B shape, 256 x 128 tile) against 148 unaligned.
EXTRA = {"gemm.hip": ["-Xarch_device", "-falign-loops=128"]}


def _compile(src):
    obj = os.path.join(HERE, "_build", os.path.splitext(src)[0] + ".o")
    os.makedirs(os.path.dirname(obj), exist_ok=True)
    cmd = ["hipcc", *FLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "is not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose=True):
    with ThreadPoolExecutor(max_workers=6) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
