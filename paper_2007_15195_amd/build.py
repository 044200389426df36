"""Build libvecchia.so (HIP for gfx950) in-tree.

    python -m paper_2007_15195_amd.build          # or build() from Python

Every source under csrc/ is compiled with hipcc for --offload-arch=gfx950 and
linked into paper_2007_15195_amd/_lib/libvecchia.so. Packed FP32 instructions
are disabled for the device code (-packed-fp32-ops).
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIBDIR = os.path.join(HERE, "_lib")
LIB = os.path.join(LIBDIR, "libvecchia.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

SOURCES = [
    "kernels_plan.hip",
    "kernels_setup.hip",
    "kernels_qmc.hip",
    "kernels_qmc_f32.hip",
    "kernels_qmc_f32_long.hip",
    "kernels_qmc_f32_block.hip",
    "kernels_qmc_f64.hip",
    "kernels_qmc_f64_long.hip",
    "kernels_finalize.hip",
    "runtime.cpp",
    "server.cpp",
    "api.cpp",
    "host_order.cpp",
    "autotune.cpp",
    "calibrate.hip",
    "mixture.cpp",
    "fullsov.hip",
    "probe.hip",
    "noalloc.hip",
]

COMMON = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-Wall", "-Wno-unused-function",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-I", CSRC, "-I", os.path.join(os.path.dirname(HERE), "include")]


# Per-file flags. fullsov.hip: MFMA accumulators stay in VGPRs (gfx950 takes
# them there), so the product loop carries no accumulator copies; and constants
# are not hoisted out of the loops over dimensions, where they would take the
# registers of the recursion and be reloaded from scratch memory at every step.
EXTRA = {"fullsov.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form", "-mllvm", "-disable-machine-licm"]}


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [HIPCC, *COMMON, *EXTRA.get(src, []), "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    os.makedirs(LIBDIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
