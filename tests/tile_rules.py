"""The launchers' tile rules (csrc/tile_rules.h) compiled for the host, so that
tests can say which tile a size takes."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_11136_amd", "csrc")

SHIM = r"""
#include "tile_rules.h"
using namespace xema;
extern "C" {
int gemm_main() { return GEMM_MAIN; }
int gemm(long long M, int N, int K, int heads_dim, long long* split) {
  const GemmPick p = gemm_pick(M, N, K, heads_dim);
  *split = p.split;
  return p.tile;
}
int upconv_count() { return kNumUpconvTiles; }
int upconv(int n, int h, int w, int ci, int co, int row_begin, int row_count) {
  return upconv_pick(UpconvSize{n, h, w, ci, co, row_begin, row_count});
}
}
"""


@functools.lru_cache(None)
def lib() -> ctypes.CDLL:
    with tempfile.TemporaryDirectory(prefix="tile_rules_") as d:
        src, so = os.path.join(d, "shim.cpp"), os.path.join(d, "shim.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, src, "-o", so], check=True)
        return ctypes.CDLL(so)


GEMM_TILES = ("256x192", "256x128", "128x192", "128x128", "128x96", "64x128", "64x64")


def gemm(M, N, K, heads_dim=0):
    """The tile as "rows x columns"; for the 256-column tiles "256x256", "128x256" or both joined by "+", as they
    divide the rows."""
    split = ctypes.c_longlong()
    t = lib().gemm(ctypes.c_longlong(M), N, K, heads_dim, ctypes.byref(split))
    if t < lib().gemm_main():
        return GEMM_TILES[t]
    return "+".join(["256x256"] * (split.value > 0) + ["128x256"] * (split.value < M))


def upconv(n, h, w, ci, co, row_begin=0, row_count=None) -> int:
    return lib().upconv(n, h, w, ci, co, row_begin, h if row_count is None else row_count)
