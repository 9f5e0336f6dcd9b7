"""The attention kernels with fewer queries a workgroup, which launches that do
not fill the GPU take: against fp64, and bit for bit against the kernel the
same queries take in a larger or smaller call."""
import math

import pytest
import torch

import paper_2607_11136_amd as X
from gpu_util import DEV

pytestmark = pytest.mark.gpu

# (head_dim, heads, tokens, query ranges): the ranges reach the kernels of 512, 256 and 128 queries at head_dim 64 and
# of 256 and 128 at 128, with a first, a last and ragged ranges
CASES = [
    (64, 48, 2100, ((0, 2100), (0, 1), (2099, 1), (37, 128), (500, 129), (64, 700), (1000, 1100), (1, 1023))),
    (128, 24, 2641, ((0, 2641), (0, 1), (2640, 1), (37, 128), (500, 129), (64, 1000), (600, 1500))),
    (64, 4, 70, ((0, 70), (3, 33))),
    (128, 4, 64, ((0, 64), (63, 1))),
    (64, 2, 1, ((0, 1),)),
]


@pytest.mark.parametrize("d,H,L,ranges", CASES)
def test_query_ranges_agree(d, H, L, ranges):
    print(f"attention d={d} heads={H} tokens={L}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(d + L)
    Lp = X.padded_len(L)

    def rows(scale):
        z = torch.zeros((H, Lp, d), device=DEV)
        z[:, :L] = torch.randn((H, L, d), generator=g, device=DEV) * scale
        return z.half()

    q, k, v = rows(math.log2(math.e) / math.sqrt(d)), rows(1.0), rows(1.0)
    q[:, ::5] *= 6      # some queries' scores grow far enough to move the reference max at later tiles
    vt = v.transpose(1, 2).contiguous()

    def run(q0, n):
        o = torch.full((n + 1, H * d), float("nan"), dtype=torch.float16, device=DEV)
        X.xema_op_attention(q, k, vt, 1, H, d, L, Lp, q0, n, o)
        torch.cuda.synchronize()
        assert torch.isnan(o[n]).all(), "wrote past the last query"
        return o[:n]

    full = run(*ranges[0])
    for h in {0, H - 1}:
        s = q[h, :L].double() @ k[h, :L].double().t() * math.log(2)
        ref = torch.softmax(s, -1) @ v[h, :L].double()
        err = (full[:, h * d:(h + 1) * d].double() - ref).abs()
        # fp16 P (2^-11 of weights that sum to 1, against |v| < 6), one fp16 rounding of the result
        assert (err <= 6 * 2.0 ** -11 + 2.0 ** -10 * ref.abs()).all(), float(err.max())
    for q0, n in ranges[1:]:
        assert torch.equal(run(q0, n), full[q0:q0 + n]), (q0, n)
