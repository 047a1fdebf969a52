"""Build liblidkrylov.so (HIP kernels + C ABI) in-tree for gfx950.

    python -m paper_1704_08521_amd.build        (or: python paper_1704_08521_amd/build.py)
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "liblidkrylov.so")
SOURCES = ["lk_stencil.hip", "lk_transform.hip", "lk_m4.hip", "lk_mx.hip", "lk_kernels.hip", "lk_nn.hip", "lk_api.cpp", "lk_krylov.cpp",
           "lk_linalg.cpp", "lk_nn_host.cpp", "lk_planes.hip", "lk_planes_host.cpp",
           "lk_tpt.hip", "lk_modes.cpp", "lk_stokes.cpp", "lk_noalloc.hip"]
ARCH = os.environ.get("LK_OFFLOAD_ARCH", "gfx950")

# -packed-fp32-ops: never emit packed FP32 arithmetic (v_pk_*_f32)
FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc():
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False) -> str:
    hipcc = _hipcc()
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError(f"compile failed: {src}\n{res.stderr}")
        return obj

    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = OUT + ".tmp"
    cmd = [hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed\n{res.stderr}")
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
