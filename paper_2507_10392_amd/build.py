"""Builds libstage.so (hipcc, gfx950 only) in-tree next to this file."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libstage.so")
SOURCES = ["stage.hip", "ministages.hip", "ops_api.hip", "elementwise.hip", "gemm_simple.hip", "gemm_f32.hip", "gemm_small.hip", "gemm_mfma.hip", "gemm_mfma_256x256.hip",
           "gemm_mfma_256x192.hip", "gemm_mfma_256x128.hip", "gemm_mfma_128x128.hip", "gemm_mfma_256x256_f16.hip", "gemm_mfma_256x192_f16.hip", "gemm_mfma_256x128_f16.hip", "gemm_mfma_128x128_f16.hip",
           "attention_simple.hip", "attention_f32.hip", "attention_mfma.hip", "attention_mfma_f16.hip", "attention_split.hip", "attention_split_f16.hip", "mfma_rate.hip", "lds_probe.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


def _hipcc() -> str:
    for c in ("/opt/rocm/bin/hipcc", "hipcc"):
        if os.path.exists(c) or c == "hipcc":
            return c
    return "hipcc"


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compiles every translation unit and links the shared library.  Always recompiles."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    hipcc = _hipcc()

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr[-6000:]}")
        if verbose and r.stderr.strip():
            print(r.stderr, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr[-6000:]}")
    return LIB


if __name__ == "__main__":
    print(build())
