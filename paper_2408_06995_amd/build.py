"""Build libfpq.so (HIP, gfx950 only) and the binding's native calls (_fpqcall.so) in-tree.

Usage: python -m paper_2408_06995_amd.build
"""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libfpq.so")
CALLS = os.path.join(HERE, "_fpqcall.so")
OBJ = os.path.join(HERE, "_build")
SOURCES = ["api.hip", "quant.hip", "search.hip", "sparsity.hip", "rounding.hip", "gemm.hip", "gemm_dma.hip", "gemm_dma_q.hip", "gemm_dma_s.hip", "gemm_dma_sq.hip", "gemm_strip.hip", "gemm_strip_h.hip", "gemm_strip_q.hip", "gemm_wk.hip", "gemm_wk_q.hip", "gemm_wk16.hip", "gemm_wk16_h.hip", "peaks.hip", "gemm_sparse.hip", "igemm.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src):
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = ["hipcc"] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build_calls():
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-missing-field-initializers",
                           "-I", sysconfig.get_paths()["include"], os.path.join(CSRC, "pycall.cpp"), "-o", CALLS])


def build():
    os.makedirs(OBJ, exist_ok=True)
    build_calls()
    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(_compile, SOURCES))
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", OUT])
    return OUT


if __name__ == "__main__":
    print(build())
