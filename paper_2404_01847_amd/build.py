"""Builds libs24.so (the C-ABI HIP library) in-tree with hipcc for gfx950.

    python -m paper_2404_01847_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libs24.so")
OBJ = os.path.join(HERE, "_build")

SOURCES = ["s24_host.hip", "s24_mask.hip", "s24_elementwise.hip", "s24_gemm.hip", "s24_gemm_f32.hip", "s24_gemm_slice.hip", "s24_gemm_joint.hip", "s24_mvue.hip", "s24_probe.hip"]
# The command processor puts the first 14 dwords of a kernel's arguments into scalar registers before a wave starts.  Without that a wave
# begins with a trip to memory for them, which is half a microsecond of a kernel of eight (256 tokens x 768 x 3072, four sliced products:
# 51.4 -> 49.5 us a step; two of 16 tokens: 41.7 -> 40.4).  It works on numbers, pointers and vectors (not on structures), those that
# the first address needs first.
PRELOAD_ARGUMENTS = ["-mllvm", "-amdgpu-kernarg-preload-count=14"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", *PRELOAD_ARGUMENTS,
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = [_hipcc(), *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the gfx-only feature flag; that warning is harmless
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(6, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stderr)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
