"""Build librom.so (HIP, gfx950) in-tree with hipcc.

Every HIP source is compiled for gfx950 only, with packed FP32 instructions disabled,
then linked into paper_2311_03694_amd/librom.so next to this file.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "librom.so")
SOURCES = ["k_als.hip", "k_bdf.hip", "k_contract.hip", "k_dense1.hip", "k_fold.hip", "k_gemm.hip", "k_kr.hip", "k_mfma.hip", "k_multi.hip",
           "k_res.hip", "rom_api.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


# Per-source flags.  k_kr.hip, k_fold.hip and k_gemm.hip keep their MFMA accumulators in VGPRs
# (the per-j VALU weighting of k_kr and k_fold reads them every iteration; accumulators in AGPRs would need a copy
# each time, and the ring registers k_gemm needs fit beside them).
EXTRA = {"k_kr.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"], "k_fold.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
         "k_gemm.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
