"""The GEMM dispatch (csrc/gemm_route.h, host arithmetic) compiled with g++ for
the tests that need to know which kernel given sizes take (not collected by
pytest)."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2608_07974_amd", "csrc")
TILE_256, TILE_128, TILE_128_WIDE = 0, 1, 2
SPK = 4 << 20  # floats of a chunk's split-K workspace

SRC = r"""
#include "gemm_route.h"
extern "C" void route(int M, int N, int K, int ak, int bk, int may_split, size_t part_elems, int heads,
                      int hd, int dma256, int dma128, int bkt, int* out) {
  const zl::GemmShape g = {M, N, K, ak != 0, bk != 0, may_split != 0, part_elems, heads != 0, hd};
  const zl::GemmRoute r = zl::route_gemm(g, [&](int R) { return (R == 256 ? dma256 : dma128) != 0; });
  out[0] = r.tile;
  out[1] = r.dma;
  out[2] = zl::split_k(K, r.nz, bkt, out[4]);
  out[3] = zl::wave_columns(r.tile);
}
extern "C" int skinny(int M, int N, int K, int bk, size_t part_elems, int np) {
  const zl::GemmShape g = {M, N, K, true, bk != 0, part_elems > 0, part_elems, false, 0};
  const zl::GemmShape p[3] = {g, g, g};
  return zl::skinny_better(p, np);
}
extern "C" int deep(int ak, int bk, long blocks, int k) { return zl::deep_stages(ak != 0, bk != 0, blocks, k); }
extern "C" int f32_large(int M, int N, int K, int ak, int bk) {
  return zl::f32_large_tiles(M, N, K, ak != 0, bk != 0);
}
"""


@functools.lru_cache(None)
def _lib():
    d = tempfile.mkdtemp(prefix="gemm_route")
    src, so = os.path.join(d, "route.cpp"), os.path.join(d, "route.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", so],
                   check=True)
    return ctypes.CDLL(so)


def route(M, N, K, ak, bk, part_elems=SPK, may_split=True, heads=False, hd=0, dma256=True, dma128=True):
    """dict(tile, dma, nz, wave_cols, ksplit): the kernel that a bf16 GEMM of these sizes takes."""
    out = (ctypes.c_int * 5)()
    _lib().route(M, N, K, int(ak), int(bk), int(may_split), ctypes.c_size_t(part_elems), int(heads), hd,
                 int(dma256), int(dma128), 64 if ak and bk else 32, out)
    return dict(tile=out[0], dma=bool(out[1]), nz=out[2], wave_cols=out[3], ksplit=out[4])


def f32_large(M, N, K, ak, bk):
    """Whether an fp32 GEMM takes the 64 x 64 tiles."""
    return bool(_lib().f32_large(M, N, K, int(ak), int(bk)))


def skinny(M, N, K, bk, part_elems=SPK, np=1):
    """Whether np products of few columns over a K-major A take whole rows per block."""
    return bool(_lib().skinny(M, N, K, int(bk), ctypes.c_size_t(part_elems), np))


def deep(ak, bk, blocks, k):
    """Whether 128 x 128 tiles keep 256 of K in flight."""
    return bool(_lib().deep(int(ak), int(bk), ctypes.c_long(blocks), k))
