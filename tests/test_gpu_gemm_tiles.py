"""Every tile of the GEMM against fp64, and against each other bit for bit: the
tile is picked from the problem's size, so the same rows computed in a smaller
call take other tiles and must give the same bytes."""
import math

import pytest
import torch

import paper_2607_11136_amd as X
import workloads as W
from gpu_util import DEV, Device, slot_view

pytestmark = pytest.mark.gpu

EPI = {"bias": X.XEMA_EPI_BIAS, "gelu": X.XEMA_EPI_BIAS_GELU, "gated": X.XEMA_EPI_GATED_RESIDUAL}


def _gelu(u):
    return 0.5 * u * (1 + torch.tanh(math.sqrt(2 / math.pi) * (u + 0.044715 * u ** 3)))


# N, K and the row counts of each reach every tile of the rule and both heights of the 256-column tiles, alone and
# together (a CPU test asserts it); each count has a neighbour at the tile's edge and a ragged last tile
ROWS = (1, 63, 65, 128, 129, 511, 513, 1000, 1025, 2047, 4095, 6001)
SIZES = ((3072, 192), (4096, 64), (768, 320))
M_FULL = 9216


@pytest.mark.parametrize("N,K", SIZES)
@pytest.mark.parametrize("dtype,epi", [("f16", "gelu"), ("f16", "gated"), ("bf16", "bias"), ("bf16", "gelu"), ("bf16", "gated")])
def test_tiles_agree(N, K, dtype, epi):
    code, t = (X.XEMA_F16, torch.float16) if dtype == "f16" else (X.XEMA_BF16, torch.bfloat16)
    g = torch.Generator(device=DEV).manual_seed(N + K)
    M = M_FULL
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


# (head_dim, hidden, tokens): the QKV GEMM of the whole sequence takes the tiles of its epilogue at each head width
# (asserted on the CPU), that of 60-token chunks the smallest
HEADS = [(64, 256, 200), (64, 256, 1600), (64, 512, 1613), (64, 256, 8200), (64, 512, 4001), (64, 512, 8209),
         (128, 256, 200), (128, 512, 1613), (128, 256, 8200), (128, 512, 4001), (128, 512, 8209)]


@pytest.mark.parametrize("d,D,L", HEADS)
def test_qkv_heads_agree(d, D, L):
    """Q, K and V^T of a block run at once and in small chunks, with every value finite."""
    print(f"qkv d={d} hidden={D} tokens={L}", flush=True)
    s = W.tiny_shape(name="qkv", cfg_id=70, batch=1, text_len=3, grid=(1, 1, L - 3), hidden=D, heads=D // d, head_dim=d,
                     mlp_hidden=256, cond_dim=256, rope_dims=(0, 0, d // 2))
    dev = Device(W.make_inputs(s))
    Lp, H = X.padded_len(L), D // d
    got = []
    for chunk in (0, 60):
        _, ws, plan = dev.run(chunk)
        got.append([slot_view(ws, plan, n, torch.float16, (H, Lp, d)).clone() for n in ("q", "k", "vt")])
    for a, b in zip(*got):
        assert torch.isfinite(a).all() and torch.equal(a.view(torch.int16), b.view(torch.int16))
