"""The rules by which the launchers pick a tile, on the host: the GPU tests reach
every tile they are meant for, and what a rule picks fits the kernel's limits."""
import random

import pytest

import test_gpu_gemm_tiles as GT
import test_gpu_vae_tiles as VT
import tile_rules as T


def test_vae_shapes_reach_every_tile():
    tiles = set(range(T.lib().upconv_count()))
    assert {T.upconv(*s) for s in VT.SHAPES} == tiles
    assert {T.upconv(*s) for s, _ in VT.NAN_PIXELS} == tiles


@pytest.mark.parametrize("seed", range(4))
def test_vae_flat_tiles_only_where_x_fits(seed):
    """A tile of corners in a row holds x of its corners and of a row and two pixels more, beside three units of
    weights in 160 KB of LDS, and its outputs within 2^31 bytes."""
    rng = random.Random(seed)
    for _ in range(2000):
        n, h, w = rng.randint(1, 64), rng.choice((1, 2, rng.randint(1, 600))), rng.choice((1, rng.randint(1, 1000)))
        ci, co = 64 * rng.randint(1, 8), 256 * rng.choice((1, 2, 4, 64))
        rc = rng.choice((h, rng.randint(1, h)))
        t = T.upconv(n, h, w, ci, co, rng.randint(0, h - rc), rc)
        groups, corners = {3: (4, 192), 4: (8, 256), 5: (8, 128)}.get(t, (0, 0))
        if corners:
            x_rows = -(-(corners + w + 2) // 8) * 8
            assert 2 * 128 * x_rows + 3 * 7 * 128 * (128 // groups) <= 160 * 1024
            frames = corners // ((rc + 1) * (w + 1)) + 2
            assert frames * 8 * h * w * co < 2 ** 31


def test_gemm_sizes_reach_every_tile():
    got = {T.gemm(m, n, k) for n, k in GT.SIZES for m in (*GT.ROWS, GT.M_FULL)}
    assert got == {*T.GEMM_TILES, "256x256", "128x256", "256x256+128x256"}


def test_qkv_sizes_reach_every_tile_of_their_epilogue():
    main = {"256x256", "128x256", "64x128", "128x128", "256x128"}
    for d, tiles in ((64, main | {"64x64"}), (128, main)):
        assert {T.gemm(l, 3 * h, h, d) for e, h, l in GT.HEADS if e == d} == tiles
        assert T.gemm(60, 768, 256, d) == T.gemm(60, 1536, 512, d) == ("64x64" if d == 64 else "64x128")


@pytest.mark.parametrize("seed", range(4))
def test_gemm_rule_keeps_to_the_kernels_limits(seed):
    """Every pick divides N, the QKV epilogue gets two waves a row of heads, and the split is a tile boundary."""
    rng = random.Random(seed)
    for _ in range(2000):
        M, N, K = rng.randint(1, 30000), 256 * rng.randint(1, 48), 64 * rng.randint(1, 192)
        heads = rng.choice((0, 64, 128))
        t = T.gemm(M, N, K, heads)
        for part in t.split("+"):
            assert N % int(part.split("x")[1]) == 0
        if heads:
            assert t in ("64x128", "128x128", "256x128") or t.endswith("x256") or (heads, t) == (64, "64x64")
