"""The upsampling stage at the edges of its tiles: each of the six tiles (a CPU
test says that SHAPES reach them), images of one pixel up to a few tiles, one and
several K steps and rounds of tiles, against fp64; row bands, which take other
tiles, bit for bit; a NaN pixel, which reaches the outputs that see it and no other;
and weights whose summed taps differ widely in size."""
import pytest
import torch

import paper_2607_11136_amd as X
from gpu_util import DEV

pytestmark = pytest.mark.gpu

SHAPES = [
    (1, 1, 1, 64, 256),      # one pixel
    (2, 8, 15, 64, 256),
    (30, 7, 16, 128, 256),   # two rounds of tiles
    (16, 10, 16, 128, 256),
    (20, 16, 33, 192, 256),  # four rounds
    (16, 12, 16, 64, 256),
    (24, 15, 33, 64, 256),   # three rounds, one K step
    (1, 31, 46, 64, 512),
    (3, 15, 130, 192, 256),  # 16 x 16 corners a tile, one row and two columns past the last
    (1, 13, 223, 128, 256),  # 12 x 16
    (1, 13, 300, 128, 256),  # 4 x 48
]


def stage(shape, bad=None, scale=None):
    n, h, w, ci, co = shape
    g = torch.Generator(device=DEV).manual_seed(sum(shape))
    x = torch.randn((n, h, w, ci), generator=g, device=DEV).bfloat16()
    wt = (torch.randn((co, 3, 3, ci), generator=g, device=DEV) / (9 * ci) ** 0.5).bfloat16()
    b = torch.randn((co,), generator=g, device=DEV).bfloat16()
    if bad:
        x[bad] = float("nan")
    if scale:
        scale(x, wt, b)
    wp = torch.empty(X.xema_vae_upconv_weight_bytes(ci, co), dtype=torch.uint8, device=DEV)
    X.xema_vae_upconv_prepare(wt, ci, co, wp)

    def run(r0, rc):
        y = torch.full((n, 2 * h, 2 * w, co), 7.0, dtype=torch.bfloat16, device=DEV)
        X.xema_vae_upconv(x, n, h, w, ci, wp, b, co, r0, rc, y)
        torch.cuda.synchronize()
        return y
    return x, wt, b, run


@pytest.mark.parametrize("shape", SHAPES)
def test_tiles_match_definition(shape):
    print(f"vae {shape}", flush=True)
    n, h, w, ci, co = shape
    x, wt, b, run = stage(shape)
    up = x.double().repeat_interleave(2, 1).repeat_interleave(2, 2)
    up = torch.nn.functional.pad(up, (0, 0, 1, 1, 1, 1))
    ref = b.double().expand(n, 2 * h, 2 * w, co).clone()
    for ky in range(3):
        for kx in range(3):
            ref += up[:, ky:ky + 2 * h, kx:kx + 2 * w] @ wt[:, ky, kx].double().t().contiguous()
    y = run(0, h)
    # one bf16 rounding (8 significant bits: half an ulp is at most 2^-8 of the value), the summed weights to 2^-17
    # and fp32 sums of unit size
    err = (y.double() - ref).abs()
    assert (err <= 2.0 ** -8 * ref.abs() * 1.01 + 2e-4).all(), float(err.max())
    for r0, rc in {(0, 1), (h - 1, 1), (h // 2, h - h // 2), (h // 3, max(h // 3, 1)), (max(h - 8, 0), min(h, 8))}:
        band = run(r0, rc)
        assert torch.equal(band[:, 2 * r0:2 * (r0 + rc)], y[:, 2 * r0:2 * (r0 + rc)]), (r0, rc)
        assert (band[:, :2 * r0] == 7).all() and (band[:, 2 * (r0 + rc):] == 7).all(), (r0, rc)


# pixels at the tiles' corners, at the borders of waves inside a tile, and at the images' edges
NAN_PIXELS = [
    ((1, 31, 46, 64, 256), (0, 0, 0)),
    ((1, 31, 46, 64, 256), (0, 15, 15)),
    ((1, 31, 46, 64, 256), (0, 16, 31)),
    ((1, 31, 46, 64, 256), (0, 30, 45)),
    ((3, 15, 130, 192, 256), (1, 3, 15)),
    ((3, 15, 130, 192, 256), (1, 4, 16)),
    ((3, 15, 130, 192, 256), (2, 14, 129)),
    ((1, 13, 223, 128, 256), (0, 11, 47)),
    ((1, 13, 223, 128, 256), (0, 12, 48)),
    ((1, 13, 300, 128, 256), (0, 3, 47)),
    ((1, 13, 300, 128, 256), (0, 12, 299)),
    ((20, 16, 33, 192, 256), (4, 15, 32)),
    ((20, 16, 33, 192, 256), (5, 0, 0)),
    ((24, 15, 33, 64, 256), (7, 7, 16)),
    ((24, 15, 33, 64, 256), (23, 14, 32)),
]


@pytest.mark.parametrize("shape,pixel", NAN_PIXELS)
def test_nan_reaches_only_its_outputs(shape, pixel):
    f, i, j = pixel
    n, h, w, ci, co = shape
    *_, run = stage(shape, bad=(f, i, j, 5))
    got = torch.isnan(run(0, h)).any(-1)
    want = torch.zeros_like(got)
    want[f, max(2 * i - 1, 0):2 * i + 3, max(2 * j - 1, 0):2 * j + 3] = True
    assert torch.equal(got, want)


def _bottom_right_taps_large(x, w, b):
    """Row 2 and column 2 of the kernel 2^12 times the others: the image's last row and column do not see them."""
    b.zero_()
    w[:, 2] *= 4096
    w[:, :, 2] *= 4096


def _top_left_taps_large(x, w, b):
    b.zero_()
    w[:, 0] *= 4096
    w[:, :, 0] *= 4096


def _taps_cancel(x, w, b):
    """Rows 0 and 1 cancel up to 2^-8, and odd rows of the image are small: half of the odd output rows consist of
    what is left of the sums of rows 0 and 1, next to rows 1 and 2 that are not small."""
    b.zero_()
    w[:, 0] = (-w[:, 1].float() * (1 - 2.0 ** -8)).bfloat16()
    x[:, 1::2] *= 2.0 ** -14


@pytest.mark.parametrize("scale", [_bottom_right_taps_large, _top_left_taps_large, _taps_cancel])
@pytest.mark.parametrize("shape", [(1, 9, 17, 64, 256), (24, 15, 33, 64, 256), (2, 15, 223, 192, 256)])
def test_sums_keep_their_own_precision(shape, scale):
    """Every output carries the summed weights it is made of to 2^-17 of their own size, however large the other
    sums of the same taps are (xema_vae.h): no output comes from a difference of larger products."""
    print(f"vae {shape} {scale.__name__}", flush=True)
    n, h, w, ci, co = shape
    x, wt, b, run = stage(shape, scale=scale)
    pad = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
    wd = wt.double()
    rows = {0: ((0,), (1, 2)), 1: ((0, 1), (2,))}
    ref = torch.zeros((n, 2 * h, 2 * w, co), dtype=torch.float64, device=DEV)
    size = torch.zeros_like(ref)           # the sum of |weight| |x| over the output's own four sums
    for py in (0, 1):
        for px in (0, 1):
            for a in (0, 1):
                for c in (0, 1):
                    s = sum(wd[:, ky, kx] for ky in rows[py][a] for kx in rows[px][c]).t().contiguous()
                    z = pad[:, py + a:py + a + h, px + c:px + c + w]
                    ref[:, py::2, px::2] += z @ s
                    size[:, py::2, px::2] += z.abs() @ s.abs()
    # the weights' hi + lo; fp32 sums of up to 7 ci products, each addition to 2^-24 of what is summed; one bf16 rounding
    err = (run(0, h).double() - ref).abs()
    tol = (2.0 ** -17 + 7 * ci * 2.0 ** -24) * size + 2.0 ** -8 * ref.abs()
    assert (err <= tol).all(), float((err / tol).max())
