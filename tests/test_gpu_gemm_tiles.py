"""Every tile of the GEMM against fp64, and against each other bit for bit: the
tile is picked from the problem's size, so the same rows computed in a smaller
call take other tiles and must give the same bytes."""
import math

import pytest
import torch

import paper_2607_11136_amd as X
from gpu_util import DEV

pytestmark = pytest.mark.gpu

EPI = {"bias": X.XEMA_EPI_BIAS, "gelu": X.XEMA_EPI_BIAS_GELU, "gated": X.XEMA_EPI_GATED_RESIDUAL}


def _gelu(u):
    return 0.5 * u * (1 + torch.tanh(math.sqrt(2 / math.pi) * (u + 0.044715 * u ** 3)))


# N = 3072 reaches the tiles 64 x 64, 64 x 128, 128 x 96, 128 x 128, 128 x 192, 256 x 192 and 256 x 256 with these
# row counts, N = 4096 also 256 x 128; each count has a neighbour at the tile's edge and a ragged last tile
ROWS = (1, 63, 65, 128, 129, 511, 513, 1000, 1025, 2047, 4095)


@pytest.mark.parametrize("N,K", [(3072, 192), (4096, 64)])
@pytest.mark.parametrize("dtype,epi", [("f16", "gelu"), ("f16", "gated"), ("bf16", "bias"), ("bf16", "gated")])
def test_tiles_agree(N, K, dtype, epi):
    code, t = (X.XEMA_F16, torch.float16) if dtype == "f16" else (X.XEMA_BF16, torch.bfloat16)
    g = torch.Generator(device=DEV).manual_seed(N + K)
    M = 9216                                   # 256 x 256 tiles, then half-height ones
    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV)
    a, b = normal(M, K).to(t), (normal(N, K) / math.sqrt(K)).to(t)
    bias, resid, gate = normal(N).bfloat16(), normal(M, N), normal(1, N)
    gated = epi == "gated"
    ct = torch.float32 if gated else t

    def run(rows):
        c = torch.full((rows + 1, N), float("nan"), dtype=ct, device=DEV)
        X.xema_op_gemm(X.gemm_args(code, a, rows, K, b, N, bias, EPI[epi], c, X.XEMA_F32 if gated else code, N,
                                   resid=resid, ld_resid=N if gated else 0, gate=gate))
        torch.cuda.synchronize()
        assert torch.isnan(c[rows]).all(), "wrote past the last row"
        return c[:rows]

    full = run(M)
    ref = a.double() @ b.double().t() + bias.double()
    ref = resid.double() + gate.double() * ref if gated else _gelu(ref) if epi == "gelu" else ref
    # fp32 sums of K products of unit-variance terms, then one rounding of the output type
    ulp = {torch.float32: 2.0 ** -24, torch.float16: 2.0 ** -11, torch.bfloat16: 2.0 ** -8}[ct]
    err = (full.double() - ref).abs()
    assert (err <= 2e-5 * (gate.abs().double() if gated else 1.0) + 1.5 * ulp * ref.abs() + 1e-5).all(), float(err.max())
    for rows in ROWS:
        assert torch.equal(run(rows), full[:rows]), rows
