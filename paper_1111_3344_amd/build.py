"""Compile the HIP library (libbssn_hip.so) for gfx950, in-tree.

Every translation unit is compiled to an object in parallel, then linked
with hipcc.  Packed FP32 instructions are disabled for all device code.
"""
import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libbssn_hip.so")
SOURCES = ["bssn_api.cpp", "bssn_rhs_o4.hip", "bssn_rhs_o8.hip",
           "bssn_constraints.hip", "bssn_batch.cpp",
           "bssn_batch_o4.hip", "bssn_batch_o8.hip", "bssn_radiative.hip", "bssn_adm.hip",
           "bssn_amr_plan.cpp", "bssn_amr.hip", "bssn_multipole.hip",
           "bssn_psi4.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]
# The stage kernels hold a point's working set in 256 registers per lane.
# Hoisting the stencils' and the algebra's FP64 constants out of the tile loop
# (machine LICM) would take dozens of them and spill: off for these files.  Of
# the direct kernels in them, those without a loop compile to the same code, and
# the work-list ones are faster so (mixed precision at order 8, 24 patches:
# 6.4 instead of 8.6 ms per step).
# The order-8 work-list kernels need the scheduler's exact register tracking
# as well (2% slower code, so only where it takes the last spills away).
STAGE_FLAGS = ["-mllvm", "-disable-machine-licm"]
EXTRA_FLAGS = {
    "bssn_rhs_o4.hip": STAGE_FLAGS,
    "bssn_rhs_o8.hip": STAGE_FLAGS,
    "bssn_batch_o4.hip": STAGE_FLAGS,
    "bssn_batch_o8.hip": STAGE_FLAGS + ["-mllvm",
                                        "-amdgpu-use-amdgpu-trackers"],
}


def _compile(src, verbose):
    out = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    lang = ["-x", "hip"] if src.endswith(".cpp") else []
    extra = EXTRA_FLAGS.get(src, [])
    cmd = ["hipcc"] + FLAGS + extra + lang + ["-c", os.path.join(CSRC, src), "-o",
                                      out]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    return out


def build(verbose=False, jobs=None):
    os.makedirs(OBJ, exist_ok=True)
    srcs = [s for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    jobs = jobs or min(len(srcs), os.cpu_count() or 4)
    with cf.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o",
           LIB + ".tmp"] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
