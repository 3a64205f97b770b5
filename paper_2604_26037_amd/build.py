"""Compile libpawfe.so for gfx950 with hipcc (in-tree, no JIT cache).

    python -m paper_2604_26037_amd.build         # always recompiles

Objects go to <repo>/_build/, the shared library to
paper_2604_26037_amd/libpawfe.so.  Every HIP translation unit is built with
the packed-FP32 instructions disabled (the v_pk_*_f32 family is not used).
"""

from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libpawfe.so")

SOURCES = ["builder.cpp", "kernels_cell.hip", "kernels_cell_mfma.hip", "kernels_cell_valu.hip",
           "kernels_cell_gen_f32.hip", "kernels_cell_gen_f64.hip", "kernels_cell_step.hip",
           "kernels_cell_step_gen.hip", "kernels_nl.hip", "kernels_halo.hip", "api.hip", "batch.cpp"]
# compiled once per data type (-DPAWFE_T), the longest first: the cell kernels
# are most of the build
PER_TYPE = ["kernels_cell_valu.hip", "kernels_cell_step.hip", "kernels_cell_step_gen.hip"]
UNITS = [(s, t) for t in ("double", "float") for s in PER_TYPE] + [(s, None) for s in SOURCES if s not in PER_TYPE]
ARCH = os.environ.get("PAWFE_OFFLOAD_ARCH", "gfx950")


def hipcc():
    for cand in (os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc"), shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def _flags():
    return [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-I", INCLUDE, "-I", CSRC, "-Wno-unused-command-line-argument"]


def _object(unit):
    src, dtype = unit
    return os.path.join(BUILD, os.path.splitext(src)[0] + (f"_{dtype}" if dtype else "") + ".o")


def _compile(unit):
    src, dtype = unit
    obj = _object(unit)
    cmd = [hipcc()] + _flags() + ([f"-DPAWFE_T={dtype}"] if dtype else []) + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose=True):
    os.makedirs(BUILD, exist_ok=True)
    jobs = min(len(UNITS), int(os.environ.get("MAX_JOBS", "8")))
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, UNITS))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs + \
        ["-L", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "lib"),
         "-lrocsolver", "-lrocblas", "-Wl,-rpath," + os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "lib")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
