"""The rules by which the launchers pick a tile, on the host: the GPU tests reach
every tile they are meant for, and what a rule picks fits the kernel's limits."""
import random

import pytest

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
