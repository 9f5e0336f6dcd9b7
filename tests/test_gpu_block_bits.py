"""The block's Q, K, V^T and output keep their bits: the digests in
tests/golden/block_digests.json pin the order of every sum (the QK-RMSNorm's
over a head's columns above all) for whichever tile a size takes, so that a
program's results do not move when only the library is exchanged."""
import hashlib
import json
import os

import pytest
import torch

import paper_2607_11136_amd as X
import workloads as W
from gpu_util import Device, slot_view

pytestmark = pytest.mark.gpu

with open(os.path.join(os.path.dirname(__file__), "golden", "block_digests.json")) as _f:
    DIGESTS = json.load(_f)

SHAPES = {s.name: s for s in (
    W.TINY,
    W.tiny_shape(name="d64_b2", cfg_id=50, batch=2, text_len=45, grid=(3, 9, 23), hidden=512, heads=8, head_dim=64,
                 mlp_hidden=2048, cond_dim=512, rope_dims=(16, 24, 24)),
    W.tiny_shape(name="d128_b3", cfg_id=52, batch=3, text_len=7, grid=(5, 6, 11), hidden=768, heads=6, head_dim=128,
                 mlp_hidden=1024, cond_dim=768, rope_dims=(32, 48, 48)),
    W.IMAGE, W.VIDEO)}


def digests(s):
    out, ws, plan = Device(W.make_inputs(s)).run()
    B, Lp, H, d = s.batch, X.padded_len(s.seq_len), s.heads, s.head_dim
    parts = {n: slot_view(ws, plan, n, torch.int16, (B, H, Lp, d)) for n in ("q", "k", "vt")}
    parts["out"] = out
    return {n: hashlib.sha256(t.contiguous().view(torch.uint8).cpu().numpy().tobytes()).hexdigest()
            for n, t in parts.items()}


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_block_keeps_its_bits(name):
    print(f"block {name}", flush=True)
    assert digests(SHAPES[name]) == DIGESTS[name]
