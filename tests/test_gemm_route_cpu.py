"""Which kernel a bf16 GEMM takes, by its sizes (host code, no GPU)."""
import itertools

import pytest

from tests.gemm_route import SPK, TILE_128, TILE_256, deep, f32_large, route, skinny


@pytest.mark.parametrize("hd", [16, 32, 64, 128])
def test_rope_and_delta_tiles_hold_whole_heads(hd):
    """The RoPE and delta epilogues read a head's columns from one wave tile:
    its width is a multiple of the head size for every size, layout and copy
    path, the register-staged kernel's (operands the direct copies cannot
    reach) among them."""
    for M, heads, K in itertools.product((1, 100, 128, 600, 2100, 16384), (1, 8, 48, 1024), (64, 2048, 8192)):
        for ak, bk, d256, d128, part in itertools.product((0, 1), (0, 1), (0, 1), (0, 1), (0, SPK)):
            r = route(M, heads * hd, K, ak, bk, part, part > 0, True, hd, d256, d128)
            assert r["wave_cols"] % hd == 0, (M, heads, K, ak, bk, d256, d128, r)
            assert r["dma"] or r["nz"] == 1
            assert r["dma"] <= (d256 if r["tile"] == TILE_256 else d128)


@pytest.mark.parametrize("ak,bk", [(1, 1), (1, 0), (0, 0), (0, 1)])
def test_splits_cover_k_within_the_workspace(ak, bk):
    """Every split but the last is ksplit deep, the last is not empty, ksplit is
    a whole number of k tiles, and the partials fit."""
    bkt = 64 if ak and bk else 32
    for M, N, K, part in itertools.product((8, 200, 1000, 4096), (72, 768, 3072), (8, 520, 3000, 14336, 128256),
                                           (0, 5000, SPK)):
        r = route(M, N, K, ak, bk, part, part > 0)
        assert r["nz"] >= 1 and (r["nz"] - 1) * r["ksplit"] < K <= r["nz"] * r["ksplit"]
        if r["nz"] > 1:
            assert r["ksplit"] % bkt == 0 and r["nz"] * M * N <= part
    assert route(8192, 8192, 4096, ak, bk)["tile"] == TILE_256
    assert route(128, 128, 256, ak, bk, 0, False)["tile"] == TILE_128


def test_fp32_tiles_by_size():
    """Launches that fill the chip take the large fp32 tiles, sooner where K
    pads its tiles of 128 (1.7 - 4.8 times faster there); the small shapes of
    the fp32 configuration, and weight gradients with full K, never do."""
    for M, N, K in ((4096, 4096, 2048), (4096, 4096, 16), (2048, 2048, 64), (4096, 2048, 512)):
        assert f32_large(M, N, K, 1, 1), (M, N, K)
    assert f32_large(4096, 4096, 16, 0, 0) and f32_large(4096, 4096, 2048, 1, 0)
    for ak, bk in ((1, 1), (1, 0), (0, 0), (0, 1)):
        for M, N, K in ((128, 256, 64), (256, 256, 8), (512, 512, 1024), (1, 1, 1), (64, 64, 0)):
            assert not f32_large(M, N, K, ak, bk), (M, N, K)
    assert not f32_large(8192, 8192, 2048, 0, 0)


@pytest.mark.parametrize("M,N,K,bk,part,rows", [
    (8, 8, 64, 1, 0, True), (1024, 8, 2048, 1, SPK, True), (4096, 16, 4096, 1, SPK, True), (8192, 8, 2048, 0, SPK, True),
    (2048, 64, 14336, 1, 0, True), (8, 8, 65536, 0, 0, True), (32768, 8, 64, 1, SPK, True),
    # long K that tiles can split, or many rows of 64 columns: two to eight times
    # slower as whole rows per block
    (512, 64, 65536, 1, SPK, False), (8, 64, 14336, 1, SPK, False), (200, 32, 14336, 0, SPK, False),
    (2048, 16, 65536, 0, SPK, False), (8192, 64, 14336, 0, SPK, False), (16384, 64, 4096, 1, 0, False),
    (16384, 64, 2048, 0, SPK, False)])
def test_few_columns_by_size(M, N, K, bk, part, rows):
    """The kernel for few output columns only where it measured faster than tiles."""
    assert skinny(M, N, K, bk, part) == rows


def test_few_columns_of_several_products():
    """Products that share a launch count once for its latency, and each for its rows."""
    assert skinny(1024, 8, 8192, 0, SPK, 2) and skinny(1024, 24, 2048, 0, SPK, 3)
    assert not skinny(16384, 64, 14336, 0, SPK, 2)


def test_from_240_large_tiles_up_tiles_are_large():
    """Small tiles there only where the last round of large ones is nearly empty,
    or half empty at a short K."""
    small = {20: (64, 256, 768, 2048, 8192), 24: (64, 256), 35: (64, 256, 768), 40: (64, 256, 768)}
    for ak, bk in ((1, 1), (1, 0), (0, 0)):
        for m in (15, 16, 20, 24, 25, 28, 35, 40, 42, 48):  # x 16 large tiles: 240 ... 768
            for K in (64, 256, 768, 2048, 8192):
                r = route(256 * m, 4096, K, ak, bk)
                assert r["nz"] == 1
                assert (r["tile"] == TILE_128) == (K in small.get(m, ())), (m, K)
        assert route(80, 128256, 2048, ak, bk, 0, False)["tile"] == TILE_128  # half of a large tile is padding


def test_stages_by_k_and_blocks():
    """The deep pipeline with K-major operands, and with others only for a long
    K per block, or where the blocks together load the memory."""
    for ak, bk in ((1, 1), (1, 0), (0, 0)):
        assert not deep(ak, bk, 257, 65536) and deep(ak, bk, 16, 8192)
        for blocks, k in ((1, 64), (32, 768), (96, 2048), (144, 1500), (128, 2048), (256, 1024)):
            assert deep(ak, bk, blocks, k) == (ak and bk), (blocks, k)
        for blocks, k in ((144, 3000), (128, 4096), (256, 2048)):
            assert deep(ak, bk, blocks, k)
