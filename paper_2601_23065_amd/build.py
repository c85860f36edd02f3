"""Builds libeag.so (HIP, gfx950) in-tree with hipcc.

Every source under csrc/ is compiled as HIP for gfx950 with packed-FP32
instruction selection disabled, then linked into one shared library next to
this file. Run `python -m paper_2601_23065_amd.build` or call build().
"""
import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libeag.so")
SOURCES = ["eag_api.cpp", "eag_build.hip", "eag_trace.hip", "eag_render.hip", "eag_backward.hip", "eag_pt.hip",
           "eag_edit.hip", "eag_serve.cpp", "eag_bake.hip", "eag_stage0.hip", "eag_geom.hip", "eag_nee.hip",
           "eag_prim.hip"]

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
ARCH = os.environ.get("EAG_OFFLOAD_ARCH", "gfx950")
CFLAGS = ["-x", "hip", f"--offload-arch={ARCH}", "-O3", "-fPIC", "-std=c++17", "-Wall", "-Wno-unused-function",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _compile(src):
    path = os.path.join(CSRC, src)
    if not os.path.exists(path):
        return None
    obj = os.path.join(OBJ, src + ".o")
    cmd = [HIPCC, *CFLAGS, "-c", path, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    jobs = min(8, os.cpu_count() or 4)
    with ThreadPoolExecutor(jobs) as ex:
        objs = [o for o in ex.map(_compile, SOURCES) if o]
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
