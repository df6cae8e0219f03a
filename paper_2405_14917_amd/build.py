"""Builds libslim.so (the C-ABI library of hand-written gfx950 kernels) in-tree with hipcc."""
from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libslim.so")
OBJ_DIR = os.path.join(HERE, "_build")

SOURCES = ["ctx.hip", "util.hip", "dgemm.hip", "rgemm.hip", "gram.hip", "inverse.hip", "salience.hip", "sba.hip", "quant.hip",
           "pack.hip", "dequant.hip", "dequant_few.hip", "dequant_gemm.hip", "handover.hip", "int8_products.hip", "lwc.hip"]

# packed-fp32 code generation is switched off for all device code (a device-compiler option; the host
# pass does not know the feature and says so, which is harmless)
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-I" + INCLUDE, "-I" + CSRC,
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


# The fp64 GEMM keeps its 128 accumulator registers in ordinary VGPRs (MFMA "VGPR form"): without this the
# compiler shuttles them between the two register files on every K slab and halves the occupancy.
EXTRA_FLAGS = {"dgemm.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
               "sba.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form", "-Wno-inline-asm"],
               "int8_products.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form", "-Wno-inline-asm"],
               # gram.hip and dequant_gemm.hip set M0 in inline asm (destination of its direct-to-LDS loads) and say so in the clobber
               # list, which the compiler remarks on
               "rgemm.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form", "-Wno-inline-asm"],
               "gram.hip": ["-Wno-inline-asm"], "dequant_gemm.hip": ["-Wno-inline-asm"]}


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [hipcc(), *HIPCC_FLAGS, *EXTRA_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in proc.stderr.splitlines() if noise not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = True) -> str:
    """Compiles every source for gfx950 and links paper_2405_14917_amd/libslim.so.  Always rebuilds."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as pool:
        objs = list(pool.map(_compile, SOURCES))
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("link failed:\n" + proc.stderr)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
