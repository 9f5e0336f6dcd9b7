"""The upsampling stage at the edges of its tiles: each of the three tile
heights, images of one pixel up to a few tiles, one and several K steps and
rounds of tiles, against fp64; row bands, which take other tile heights, bit
for bit; and a NaN pixel, which reaches the outputs that see it and no other."""
import pytest
import torch

import paper_2607_11136_amd as X
from gpu_util import DEV

pytestmark = pytest.mark.gpu

SHAPES = [
    (1, 1, 1, 64, 256),      # 8-row tiles: one pixel
    (2, 8, 15, 64, 256),
    (30, 7, 16, 128, 256),   # two rounds of tiles
    (16, 10, 16, 128, 256),  # 12-row tiles
    (20, 16, 33, 192, 256),  # four rounds
    (16, 12, 16, 64, 256),   # 16-row tiles
    (24, 15, 33, 64, 256),   # three rounds, one K step
    (1, 31, 46, 64, 512),
]


def stage(shape, bad=None):
    n, h, w, ci, co = shape
    g = torch.Generator(device=DEV).manual_seed(sum(shape))
    x = torch.randn((n, h, w, ci), generator=g, device=DEV).bfloat16()
    wt = (torch.randn((co, 3, 3, ci), generator=g, device=DEV) / (9 * ci) ** 0.5).bfloat16()
    b = torch.randn((co,), generator=g, device=DEV).bfloat16()
    if bad:
        x[bad] = float("nan")
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


@pytest.mark.parametrize("pixel", [(0, 0, 0), (0, 15, 15), (0, 16, 31), (0, 30, 45)])
def test_nan_reaches_only_its_outputs(pixel):
    f, i, j = pixel
    n, h, w, ci, co = shape = (1, 31, 46, 64, 256)
    *_, run = stage(shape, bad=(f, i, j, 5))
    got = torch.isnan(run(0, h)).any(-1)[0]
    want = torch.zeros_like(got)
    want[max(2 * i - 1, 0):2 * i + 3, max(2 * j - 1, 0):2 * j + 3] = True
    assert torch.equal(got, want)
