"""The library's choice of GEMM tiles as a host function: csrc/gemm_plan.h, which holds it and
no HIP code, compiled with the host compiler."""
import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_15922_amd", "csrc")
TILES = ("64x64", "128x128", "192x128", "288x128", "128x256", "192x256", "256x256", "128x128_2")
ENTRY = """#include "gemm_plan.h"
extern "C" void plan(int M, int N, int K, int fp8, int mx8, int ng, long cus, int* out) {
  const wam::GemmPlan p = wam::plan_gemm(M, N, K, fp8, mx8, ng, cus);
  out[0] = p.tile; out[1] = p.two; out[2] = p.c1;
}
extern "C" int ntiles() { return wam::NTILES; }
"""


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as tmp:
        src, so = os.path.join(tmp, "plan.cpp"), os.path.join(tmp, "plan.so")
        with open(src, "w") as f:
            f.write(ENTRY)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", so], check=True)
        L = ctypes.CDLL(so)
    assert L.ntiles() == len(TILES)
    return L


def plan(M, N, K, fp8=False, mx8=False, ng=1, cus=256):
    """(tile,) or, for two column ranges, (tile, tile of the rest, column tiles of the first)."""
    out = (ctypes.c_int * 3)()
    _lib().plan(M, N, K, int(fp8), int(mx8), ng, ctypes.c_long(cus), out)
    return (TILES[out[0]],) if out[1] < 0 else (TILES[out[0]], TILES[out[1]], out[2])
