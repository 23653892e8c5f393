"""Build the gfx950 HIP library ``libgenga.so`` in-tree with hipcc.

Every HIP source under ``csrc/`` is compiled to an object for gfx950 and the
objects are linked into one shared library next to this file.  Packed FP32
instructions are disabled for all device code."""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgenga.so")
ARCH = os.environ.get("GENGA_OFFLOAD_ARCH", "gfx950")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-result", "-I", os.path.join(HERE, "..", "include")]
# The batched kernel is instantiated for one and for two systems per wave; with
# multiply-adds fused only inside one source expression (not wherever the
# code generator finds a pair) both layouts round identically.
# The hybrid adjoint's forward map rounds like the plain FP64 definitions it
# differentiates (no fused multiply-adds), so that its close encounters follow
# theirs as closely as rounding allows.
# The BS loops of the main mode run one wave to a SIMD, whose time follows where
# their code falls in the instruction cache's lines: loops start on a line, so
# that an edit elsewhere in the kernel does not move them (777 bodies 0.990 to
# 0.994 times the speed without, 1.000 with).
FILE_FLAGS = {"batch.hip": ["-ffp-contract=on"], "hadj.hip": ["-ffp-contract=off"],
              "massive.hip": ["-falign-loops=64"]}


def _compile(src: str, obj: str) -> None:
    cmd = [HIPCC, *FLAGS, *FILE_FLAGS.get(os.path.basename(src), []), "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")


def build(verbose: bool = False) -> str:
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = [os.path.join(objdir, os.path.basename(s) + ".o") for s in srcs]
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        list(ex.map(lambda so: _compile(*so), zip(srcs, objs)))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
