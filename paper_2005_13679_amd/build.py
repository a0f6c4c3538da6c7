"""Builds libmc.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2005_13679_amd.build
"""

from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmc.so")

# (source, object, extra flags); mc_tiles.hip holds the kernels of one orbital
# count and part per compilation, the longest ones first
# The one-row kernels fuse multiplications and additions per expression, not as the
# back end sees fit: the same tile then has the same bits in every kernel it is
# compiled into (alone, in a batch's group, in a joint launch).
TILE_FLAGS = ("-ffp-contract=on",)
SOURCES = [("mc_tiles.hip", f"mc_tiles_{m}_{p}",
            (f"-DMC_TILES_M={m}", f"-DMC_TILES_PART={p}", *TILE_FLAGS))
           for m in range(8, 0, -1) for p in (3, 2, 0, 1) if p < 3 or m >= 5]
SOURCES += [("mc_joint.hip", f"mc_joint_{k}", (f"-DMC_JOINT_KIND={k}", *TILE_FLAGS)) for k in range(5)]
SOURCES += [(f"{n}.hip", n, ()) for n in
            ("mc_ops", "mc_block", "mc_block_sparse", "mc_host", "mc_tables", "mc_direct", "mc_batch", "mc_krylov",
             "mc_gram_direct", "mc_gram_tables")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-Wall",
    "-Wno-unused-function",
    "-Wno-cuda-compat",
    # packed FP32 instructions are disabled for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the compile-time stream plans (up to M = 7) take more constant-
    # evaluation steps than the default allows
    "-fconstexpr-steps=33554432",
    f"-I{INCLUDE}",
    f"-I{CSRC}",
]


def _compile(unit) -> str:
    src, name, extra = unit
    obj = os.path.join(BUILD, name + ".o")
    cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src} ({name}):\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    """Compiles every source and links libmc.so.  Always rebuilds."""
    os.makedirs(BUILD, exist_ok=True)
    jobs = min(len(SOURCES), int(os.environ.get("MAX_JOBS", "8")))
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
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
