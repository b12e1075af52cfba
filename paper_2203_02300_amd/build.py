"""Build the gfx950 stereo library in-tree: ``libdco_stereo.so``.

Every source under ``csrc/`` is compiled by hipcc for gfx950 into an object
under ``_build/`` (in parallel), then linked into one shared library next to
this file.  Usage: ``python -m paper_2203_02300_amd.build``.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libdco_stereo.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17",
    "-ffp-contract=off",                       # every fused multiply-add is written out
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]

# Extra flags per source.  The two-stage aggregation kernel shares a SIMD
# between three wavefronts with chains of dependent LDS round trips; the
# scheduler that maximises instruction-level parallelism interleaves the
# independent chains of its two slices: the 1280x720, D = 128 frame takes
# 0.782 ms with it and 0.889 ms with the default one, with the same results
# bit for bit.  The WTA and the other batched work-list kernels are a little
# slower under it, so it is not global.  The soft path's matrix products read
# their accumulators with vector instructions right away: kept in vector
# registers instead of accumulation registers they save a move per output (the
# gradient row pass of 8 640x480 pairs, D = 64: 0.47 instead of 0.49 ms).
_MAX_ILP = ["-mllvm", "-amdgpu-sched-strategy=max-ilp"]
FILE_FLAGS = {
    "k_aggregate.hip": _MAX_ILP,
    "k_batch_agg.hip": _MAX_ILP,
    "k_soft.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
}


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC)
                  if f.endswith((".hip", ".cpp")))


def _compile(src):
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [HIPCC, "-x", "hip", *FLAGS, *FILE_FLAGS.get(os.path.basename(src), []), "-c", src,
           "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = sources()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp, *objs]
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
