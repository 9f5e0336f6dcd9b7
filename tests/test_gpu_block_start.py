"""What a block's first launch and its weight copies leave in a poisoned arena:
the AdaLN maps (against the op, byte for byte), zeros for every padding token
of Q, K and V^T, cleared range flags and the fp16 weights."""
import dataclasses

import pytest
import torch

import workloads as W
import paper_2607_11136_amd as X
from gpu_util import DEV, Device, poison, slot_view

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim,batch,text,grid,streams", [
    (64, 1, 0, (1, 1, 1), 1),      # one token, 63 of padding
    (64, 2, 5, (3, 5, 7), 2),
    (128, 3, 7, (1, 8, 8), 1),     # 57 of padding
    (128, 1, 0, (1, 8, 8), 2),     # no padding
])
def test_first_launch(head_dim, batch, text, grid, streams):
    d = head_dim
    s = W.BlockShape("block_start", 90 + batch, batch, text, grid, 256, 256 // d, d, 512, 256, (d // 4, d // 4, d // 4),
                     modulation_streams=streams)
    print(s, flush=True)
    dev = Device(W.make_inputs(s))
    _, ws, plan = dev.run()
    D, L, Lp, B, H = s.hidden, s.seq_len, X.padded_len(s.seq_len), batch, s.heads
    mod = slot_view(ws, plan, "mod", torch.float32, (streams, B, 6 * D))
    for i, p in enumerate(("ada", "ada_txt")[:streams]):
        want = poison(torch.empty((B, 6 * D), dtype=torch.float32, device=DEV))
        X.xema_op_adaln(dev.cond, dev.w[p + "_w"], dev.w[p + "_b"], B, s.cond_dim, 6 * D, want)
        torch.cuda.synchronize()
        assert torch.equal(mod[i], want), p
    for name in ("q", "k"):
        assert not torch.any(slot_view(ws, plan, name, torch.int16, (B, H, Lp, d))[:, :, L:])
    assert not torch.any(slot_view(ws, plan, "vt", torch.int16, (B, H, d, Lp))[..., L:])
    assert not torch.any(slot_view(ws, plan, "status", torch.int32, (X.XEMA_STATUS_WORDS,)))
    for name, w in (("wo16", "o_w"), ("wup16", "up_w"), ("wdown16", "down_w")):
        assert torch.equal(slot_view(ws, plan, name, torch.float16, tuple(dev.w[w].shape)), dev.w[w].half()), name
