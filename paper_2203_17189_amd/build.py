"""Compile the HIP sources of this package into libt5mi.so for gfx950 (in-tree, beside this file)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libt5mi.so")
OBJ_DIR = os.path.join(HERE, "_build")
SOURCES = ["relpos.hip", "rmsnorm.hip", "gemm_simple.hip", "gemm_mfma.hip", "gemm_mfma_store.hip",
           "gemm_mfma_resid.hip", "gemm_mfma_geglu_fwd.hip", "gemm_mfma_geglu_bwd.hip", "gemm_mfma_split.hip",
           "gemm_mfma_split_grouped.hip", "gemm_mfma_direct.hip", "gemm_f32.hip", "attn_simple.hip",
           "attn_mfma.hip", "attn_f32.hip", "adafactor.hip", "probe.hip", "embed_xent.hip", "block.hip", "stack.hip"]
# -packed-fp32-ops is switched off: hand-written and compiler-made packed float32 math is avoided on
# this target.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, src.replace(".hip", ".o"))
    cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
