"""Build the HIP library libbayesvis.so for gfx950 (in-tree, no JIT cache).

Every translation unit is compiled with hipcc for --offload-arch=gfx950 and
with packed-FP32 instruction selection disabled; the objects are linked into
``paper_2504_07090_amd/libbayesvis.so``.  Run ``python -m
paper_2504_07090_amd.build`` (or ``__graft_entry__.build()``).
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libbayesvis.so")
BUILD = os.path.join(HERE, "_build")

SOURCES = ["field.hip", "synth.hip", "synth_split.hip", "synth_sep.hip", "fringe_fwd.hip", "fringe_adj.hip", "gains.hip", "filter.hip", "mapmaking.hip", "api.hip",
           "hmc.hip", "serve.hip", "mass.hip", "batch.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# MFMA operands and results in ordinary VGPRs (on gfx950 they share one
# register file with the accumulator registers): no accumulator-register reads after every MFMA chain, and no
# kernel needs more registers for it (checked per kernel, no scratch).
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-mfma-vgpr-form=1",
         "-I" + os.path.join(HERE, "..", "include")]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = [s for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = OUT + ".tmp"
    cmd = [HIPCC, "-shared", "--offload-arch=gfx950", "-fPIC", "-o", tmp, *objs, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, OUT)
    if verbose:
        print("built", OUT)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
