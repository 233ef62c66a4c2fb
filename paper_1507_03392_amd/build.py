"""Build libecrpic.so (gfx950) in-tree with hipcc.

Every HIP translation unit is compiled with no FMA contraction (so each
expression rounds in the order written), no fast-math, and without packed
FP32 instructions.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIBDIR = os.path.join(HERE, "_lib")
LIB = os.path.join(LIBDIR, "libecrpic.so")
SOURCES = ["k_particles.hip", "k_step.hip", "k_step_f32.hip", "runtime.hip", "k_coulomb.hip", "k_sort.hip", "k_partner.hip"]
ARCH = os.environ.get("ECR_OFFLOAD_ARCH", "gfx950")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

CFLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-ffp-contract=off", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    "-Wall", "-Wno-unused-function",
]

# per-file additions.  Machine LICM hoists the FP64 constants of the
# collision's log/exp/sincos out of the collision loops into ~70 VGPRs,
# doubling the pair kernel's register count and halving its occupancy.
EXTRA_FLAGS = {
    "k_coulomb.hip": ["-mllvm", "-disable-machine-licm"],
    # the fused step kernels hold the same collision loop.  Spilled VGPRs at
    # four waves per SIMD, with LICM and without: 788 and 26 in k_period, 895
    # and 12 in k_step; in binary32-mixed 286 and 3, 290 and 2
    "k_step.hip": ["-mllvm", "-disable-machine-licm"],
    "k_step_f32.hip": ["-mllvm", "-disable-machine-licm"],
}


def _compile(src, verbose):
    obj = os.path.join(LIBDIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *CFLAGS, *EXTRA_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    noise = [ln for ln in r.stderr.splitlines() if "packed-fp32-ops" not in ln and ln.strip()]
    if noise and verbose:
        print("\n".join(noise), flush=True)
    return obj


def build(verbose=False):
    os.makedirs(LIBDIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(6, len(SOURCES))) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
