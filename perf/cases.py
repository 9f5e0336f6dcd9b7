"""The work a user of this library has it do, as timed cases.

A serving program calls the block forward (one denoising-step block, whole or
in token chunks under an activation budget), the N-block step, and the VAE
decoder's upsampling stage; a program with a schedule of its own calls the
attention and GEMM steps directly.  Sizes are those of workloads/ (tiny, image,
video and long-video templates), and draw() spreads over the same ranges.
"""
import math

import torch

import paper_2607_11136_amd as X
import workloads as W

DEV = "cuda:0"
EPILOGUES = {"bias": X.XEMA_EPI_BIAS, "gelu": X.XEMA_EPI_BIAS_GELU, "gated": X.XEMA_EPI_GATED_RESIDUAL}
TYPES = {"bf16": (X.XEMA_BF16, torch.bfloat16), "f16": (X.XEMA_F16, torch.float16)}


def _block(name, s, chunk=0, weights_f16=1, streams=1):
    return {"name": name, "kind": "block", "batch": s.batch, "text": s.text_len, "gt": s.grid[0], "gh": s.grid[1],
            "gw": s.grid[2], "hidden": s.hidden, "head_dim": s.head_dim, "mlp": s.mlp_hidden, "chunk": chunk,
            "weights_f16": weights_f16, "streams": streams}


def listed():
    v = W.VAE_VIDEO
    return [
        # a request far below the sizes that fill the GPU: launches and latency
        _block("block_tiny", W.TINY, weights_f16=0),
        # one 1024 x 1024 image, weights handed over in bf16 as they are stored (head_dim 128)
        _block("block_image", W.IMAGE, weights_f16=0),
        # four images under a tight activation budget: 512-token chunks
        _block("block_image_b4_chunk", W.IMAGE_B4, chunk=512),
        # a 480 x 720, 49-frame video, the whole sequence at once (head_dim 64)
        _block("block_video", W.VIDEO),
        # the same video with dual-stream modulation, in chunks of an odd size
        _block("block_video_dual_chunk", W.VIDEO, chunk=1000, streams=2),
        # two long videos of a wider model: the largest call
        _block("block_long", W.LONG),
        # six image blocks with one block's weights streamed from host memory
        dict(_block("step_image", W.IMAGE), kind="step", blocks=6, offloaded=1),
        # the attention of one query chunk of the video
        {"name": "attention_video_chunk", "kind": "attention", "batch": 1, "heads": 48, "head_dim": 64, "keys": 17776,
         "q_begin": 12000, "q_count": 1000},
        # the attention of one image, all queries
        {"name": "attention_image", "kind": "attention", "batch": 1, "heads": 24, "head_dim": 128, "keys": 4608,
         "q_begin": 0, "q_count": 4608},
        # the out-projection of a 512-token chunk
        {"name": "gemm_out_projection_chunk", "kind": "gemm", "rows": 512, "n": 3072, "k": 3072, "type": "f16",
         "epilogue": "gated"},
        # the last upsampler of a 480 x 720 video decoder, over 8 frames
        {"name": "vae_video", "kind": "vae", "n": v.n, "h": v.h, "w": v.w, "ci": v.ci, "co": v.co, "row_begin": 0,
         "rows": v.h},
        # a band of rows of an early, low-resolution upsampler with wide channels, one image
        {"name": "vae_band", "kind": "vae", "n": 1, "h": 67, "w": 90, "ci": 512, "co": 512, "row_begin": 20, "rows": 33},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_block(rng, most):
    """A block whose algorithmic work is at most `most` FLOPs."""
    while True:
        head_dim = rng.choice((64, 128))
        hidden = rng.choice((256, 512, 1024, 1536, 2048, 3072, 4096))
        gt = rng.choice((1, 1, rng.randint(2, 16)))
        gh, gw = _log(rng, 6, 70), _log(rng, 6, 70)
        batch, text = rng.choice((1, 1, 2, 3, 4)), rng.choice((0, 77, 226, 512, rng.randint(1, 600)))
        s = W.BlockShape("", 0, batch, text, (gt, gh, gw), hidden, hidden // head_dim, head_dim, 4 * hidden, hidden, (0, 0, 0))
        if s.flops() > most or s.seq_len > 30000:
            continue
        chunk = rng.choice((0, 0, 256 * rng.randint(1, 16), rng.randint(200, 5000)))
        c = _block("", s, chunk if chunk < s.seq_len and s.seq_len <= 24 * max(chunk, 1) else 0, rng.choice((0, 1)),
                   rng.choice((1, 1, 2)))
        del c["name"]
        return c


def draw(rng):
    kind = rng.choice(("block", "block", "attention", "gemm", "vae", "vae", "step"))
    if kind == "block":
        return _draw_block(rng, 2e13)
    if kind == "step":
        c = _draw_block(rng, 2e12)
        blocks = rng.randint(2, 6)
        return dict(c, kind="step", blocks=blocks, offloaded=rng.randint(0, 1))
    if kind == "attention":
        keys = _log(rng, 64, 30000)
        q_count = min(keys, _log(rng, 32, 30000))
        return {"kind": kind, "batch": rng.choice((1, 1, 2, 4)), "heads": rng.choice((4, 12, 24, 32, 48)),
                "head_dim": rng.choice((64, 128)), "keys": keys, "q_begin": rng.randint(0, keys - q_count), "q_count": q_count}
    if kind == "gemm":
        return {"kind": kind, "rows": _log(rng, 16, 20000), "n": 256 * rng.choice((1, 4, 8, 12, 16, 36, 48)),
                "k": 64 * rng.choice((4, 16, 24, 48, 64, 192)), "type": rng.choice(("bf16", "f16")),
                "epilogue": rng.choice(("bias", "gelu", "gated"))}
    ci, co = 64 * rng.choice((2, 3, 4, 6, 8)), 256 * rng.choice((1, 1, 2))
    while True:
        n, h, w = rng.choice((1, 1, 2, rng.randint(3, 8))), _log(rng, 16, 540), _log(rng, 16, 960)
        if n * h * w * ci * co <= 8 * 240 * 360 * 256 * 256:
            break
    rows = rng.choice((h, rng.randint(1, h)))
    return {"kind": "vae", "n": n, "h": h, "w": w, "ci": ci, "co": co, "row_begin": rng.randint(0, h - rows), "rows": rows}


# -- inputs ------------------------------------------------------------------------------------------------------


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _normal(g, shape, std=1.0, mean=0.0, dtype=torch.bfloat16):
    t = torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)
    return t.mul_(std).add_(mean).to(dtype)


def _shape(c):
    d, D = c["head_dim"], c["hidden"]
    image = c["gt"] == 1
    rope = (0, d // 2, d // 2) if image else ((16, 24, 24) if d == 64 else (32, 48, 48))
    return W.BlockShape("", 0, c["batch"], c["text"], (c["gt"], c["gh"], c["gw"]), D, D // d, d, c["mlp"], D, rope,
                        modulation_streams=c["streams"], weights_f16=c["weights_f16"])


def _block_weights(g, s):
    """The workloads' distributions: N(0, 1 / fan_in), the QK gains 1 + 0.1 N(0, 1)."""
    w = {}
    for name, shape in s.weight_shapes().items():
        gain = name in ("q_gamma", "k_gamma")
        w[name] = _normal(g, shape, 0.1, 1.0) if gain else _normal(g, shape, s.fan_in(name) ** -0.5)
    if s.weights_f16:
        for name in ("o_w", "up_w", "down_w"):
            w[name] = w[name].to(torch.float16)
    return w


def _block_inputs(c, seed):
    s, g = _shape(c), _gen(seed)
    x, cond = _normal(g, (s.batch, s.seq_len, s.hidden)), _normal(g, (s.batch, s.cond_dim))
    return s, x, cond, [_block_weights(g, s) for _ in range(c.get("blocks", 1))]


def _attention_inputs(c, seed):
    """Q and K as QK-RMSNorm leaves them (with the softmax factor in Q), V of unit variance."""
    g = _gen(seed)
    B, H, d, L = c["batch"], c["heads"], c["head_dim"], c["keys"]
    Lp = X.padded_len(L)
    gain = [_normal(g, (d,), 0.1, 1.0, torch.float32) for _ in range(2)]
    out = []
    for i, scale in enumerate((math.log2(math.e) / math.sqrt(d), 1.0)):
        z = _normal(g, (B, H, L, d), dtype=torch.float32)
        z *= (z.square().mean(-1, keepdim=True) + 1e-6).rsqrt() * gain[i] * scale
        full = torch.zeros((B, H, Lp, d), dtype=torch.float16, device=DEV)
        full[:, :, :L] = z
        out.append(full)
    vt = torch.zeros((B, H, d, Lp), dtype=torch.float16, device=DEV)
    vt[..., :L] = _normal(g, (B, H, d, L), dtype=torch.float16)
    return (*out, vt)


def _gemm_inputs(c, seed):
    g = _gen(seed)
    t = TYPES[c["type"]][1]
    r, n, k = c["rows"], c["n"], c["k"]
    d = {"a": _normal(g, (r, k), dtype=t), "b": _normal(g, (n, k), k ** -0.5, dtype=t), "bias": _normal(g, (n,), k ** -0.5)}
    if c["epilogue"] == "gated":
        d["resid"], d["gate"] = _normal(g, (r, n)), _normal(g, (1, n), dtype=torch.float32)
    return d


def _vae_inputs(c, seed):
    g = _gen(seed)
    std = (9 * c["ci"]) ** -0.5
    return (_normal(g, (c["n"], c["h"], c["w"], c["ci"])), _normal(g, (c["co"], 3, 3, c["ci"]), std),
            _normal(g, (c["co"],), std))


# -- the calls ---------------------------------------------------------------------------------------------------


def prepare(case, seed):
    c, st = case, {"case": case}
    if c["kind"] in ("block", "step"):
        s, x, cond, weights = _block_inputs(c, seed)
        cfg = X.block_cfg(s.hidden, s.heads, s.head_dim, s.mlp_hidden, s.cond_dim, s.rope_dims,
                          modulation_streams=s.modulation_streams, weights_f16=s.weights_f16)
        req = X.request(s.batch, s.text_len, *s.grid)
        st.update(cfg=cfg, req=req, x=x, cond=cond, second=torch.cuda.Stream(),
                  out=torch.empty((s.batch, s.seq_len, s.hidden), dtype=torch.float32, device=DEV))
        if c["kind"] == "block":
            st["plan"] = X.xema_workspace_layout(cfg, req, c["chunk"])
            nbytes = st["plan"].workspace_bytes
        else:
            st["plan"] = X.xema_offload_plan_k(cfg, c["blocks"], c["offloaded"])
            for i in st["plan"].offloaded_blocks():
                weights[i] = {n: torch.empty(t.shape, dtype=t.dtype, pin_memory=True).copy_(t) for n, t in weights[i].items()}
            nbytes = X.xema_step_workspace_bytes(cfg, req, c["chunk"], st["plan"])
        st.update(tensors=weights, weights=[X.block_weights(w) for w in weights],
                  ws=torch.empty(nbytes, dtype=torch.uint8, device=DEV))
    elif c["kind"] == "attention":
        st["q"], st["k"], st["vt"] = _attention_inputs(c, seed)
        st["o"] = torch.empty((c["batch"] * c["q_count"], c["heads"] * c["head_dim"]), dtype=torch.float16, device=DEV)
    elif c["kind"] == "gemm":
        d = _gemm_inputs(c, seed)
        gated = c["epilogue"] == "gated"
        code, t = TYPES[c["type"]]
        st["out"] = torch.empty((c["rows"], c["n"]), dtype=torch.float32 if gated else t, device=DEV)
        st["tensors"] = d
        st["args"] = X.gemm_args(code, d["a"], c["rows"], c["k"], d["b"], c["n"], d["bias"], EPILOGUES[c["epilogue"]],
                                 st["out"], X.XEMA_F32 if gated else code, c["n"], resid=d.get("resid"),
                                 resid_dtype=X.XEMA_BF16, ld_resid=c["n"] if gated else 0, gate=d.get("gate"))
    else:
        st["x"], w, st["bias"] = _vae_inputs(c, seed)
        st["wp"] = torch.empty(X.xema_vae_upconv_weight_bytes(c["ci"], c["co"]), dtype=torch.uint8, device=DEV)
        X.xema_vae_upconv_prepare(w, c["ci"], c["co"], st["wp"])
        st["y"] = torch.zeros((c["n"], 2 * c["h"], 2 * c["w"], c["co"]), dtype=torch.bfloat16, device=DEV)
    return st


def run(st):
    c = st["case"]
    if c["kind"] == "block":
        if c["chunk"]:
            X.xema_dit_block_fwd_pipelined(st["cfg"], st["req"], st["x"], st["weights"][0], st["cond"], c["batch"],
                                           c["chunk"], st["ws"], st["ws"].numel(), st["out"], None, st["second"])
        else:
            X.xema_dit_block_fwd(st["cfg"], st["req"], st["x"], st["weights"][0], st["cond"], 0, st["ws"],
                                 st["ws"].numel(), st["out"])
        return st["out"]
    if c["kind"] == "step":
        X.xema_dit_step_fwd(st["cfg"], st["req"], st["x"], st["weights"], st["plan"], st["cond"], c["chunk"], st["ws"],
                            st["ws"].numel(), st["out"], None, st["second"])
        return st["out"]
    if c["kind"] == "attention":
        X.xema_op_attention(st["q"], st["k"], st["vt"], c["batch"], c["heads"], c["head_dim"], c["keys"],
                            st["q"].shape[2], c["q_begin"], c["q_count"], st["o"])
        return st["o"]
    if c["kind"] == "gemm":
        X.xema_op_gemm(st["args"])
        return st["out"]
    X.xema_vae_upconv(st["x"], c["n"], c["h"], c["w"], c["ci"], st["wp"], st["bias"], c["co"], c["row_begin"],
                      c["rows"], st["y"])
    return st["y"][:, 2 * c["row_begin"]:2 * (c["row_begin"] + c["rows"])]


def work(case):
    c = case
    if c["kind"] in ("block", "step"):
        s, n = _shape(c), c.get("blocks", 1)
        tokens = s.batch * s.seq_len * s.hidden
        weights = sum(math.prod(v) for v in s.weight_shapes().values())
        return {"bytes": 2 * tokens + 4 * tokens + n * 2 * weights, "flops": n * s.flops()}
    if c["kind"] == "attention":
        rows = c["batch"] * c["heads"] * c["head_dim"]
        return {"bytes": 2 * rows * (2 * c["q_count"] + 2 * c["keys"]), "flops": 4 * rows * c["q_count"] * c["keys"]}
    if c["kind"] == "gemm":
        r, n, k = c["rows"], c["n"], c["k"]
        return {"bytes": 2 * (r + n) * k + (6 if c["epilogue"] == "gated" else 2) * r * n, "flops": 2 * r * n * k}
    # every source pixel meets each of the nine taps once: the nearest upsampling repeats its products
    src = c["n"] * (min(c["h"], c["row_begin"] + c["rows"] + 1) - max(0, c["row_begin"] - 1)) * c["w"]
    return {"bytes": 2 * src * c["ci"] + 18 * c["ci"] * c["co"] + 8 * c["n"] * c["rows"] * c["w"] * c["co"],
            "flops": 18 * c["n"] * c["rows"] * c["w"] * c["ci"] * c["co"]}


def tolerance(case):
    """About four times the distance to exact(): the 16-bit roundings of the intermediates, and one of the output
    where that is 16 bits wide."""
    if case["kind"] in ("block", "step", "attention"):
        return {"rel": 1.2e-3, "max": 1e-2}
    if case["kind"] == "gemm":
        if case["epilogue"] == "gated":
            return {"rel": 1e-5, "max": 1e-4}
        return {"rel": 7e-3, "max": 4e-2} if case["type"] == "bf16" else {"rel": 1e-3, "max": 4e-3}
    return {"rel": 7e-3, "max": 4e-2}


# -- the same in 64 bits -----------------------------------------------------------------------------------------


def _softmax_rows(q, k, v):
    """softmax(q k^T) v of one head, a few rows at a time."""
    kt, step = k.t().contiguous(), max(1, (1 << 27) // k.shape[0])
    return torch.cat([torch.softmax(q[i:i + step] @ kt, -1) @ v for i in range(0, q.shape[0], step)])


def _norm(x):
    x = x - x.mean(-1, keepdim=True)
    return x / (x.square().mean(-1, keepdim=True) + 1e-6).sqrt()


def _gelu(u):
    return 0.5 * u * (1 + torch.tanh(math.sqrt(2 / math.pi) * (u + 0.044715 * u ** 3)))


def _angles(s):
    """The rotation angle of every (token, pair): axes in (t, y, w) order, none for text and the dims past them."""
    v = torch.arange(s.n_visual, device=DEV)
    _, gh, gw = s.grid
    parts = []
    for pos, dims in zip((v // (gh * gw), v // gw % gh, v % gw), s.rope_dims):
        if dims:
            j = torch.arange(dims // 2, device=DEV, dtype=torch.float64)
            parts.append(pos.double()[:, None] * s.rope_theta ** (-2 * j / dims))
    a = torch.zeros((s.seq_len, s.head_dim // 2), dtype=torch.float64, device=DEV)
    rot = torch.cat(parts, 1)
    a[s.text_len:, :rot.shape[1]] = rot
    return a


def _exact_block(s, x, cond, w):
    D, d = s.hidden, s.head_dim
    w = {n: t.double() for n, t in w.items()}
    ang = _angles(s)
    cos, sin = ang.cos(), ang.sin()

    def qk(z, gamma):
        z = z / (z.square().mean(-1, keepdim=True) + s.qk_eps).sqrt() * gamma
        a, b = z[:, 0::2], z[:, 1::2]
        return torch.stack((a * cos - b * sin, a * sin + b * cos), -1).flatten(1)

    out = []
    for b in range(s.batch):
        m = (w["ada_w"] @ cond[b] + w["ada_b"]).expand(s.seq_len, -1)
        if s.modulation_streams == 2:
            m = m.clone()
            m[:s.text_len] = w["ada_txt_w"] @ cond[b] + w["ada_txt_b"]
        shift1, scale1, gate1, shift2, scale2, gate2 = m.split(D, 1)
        h = _norm(x[b]) * (1 + scale1) + shift1
        qkv = h @ w["qkv_w"].t() + w["qkv_b"]
        o = torch.empty_like(h)
        for j in range(s.heads):
            q, k, v = (qkv[:, i * D + j * d:i * D + (j + 1) * d].contiguous() for i in range(3))
            o[:, j * d:(j + 1) * d] = _softmax_rows(qk(q, w["q_gamma"]) / math.sqrt(d), qk(k, w["k_gamma"]), v)
        x1 = x[b] + gate1 * (o @ w["o_w"].t() + w["o_b"])
        h = _norm(x1) * (1 + scale2) + shift2
        out.append(x1 + gate2 * (_gelu(h @ w["up_w"].t() + w["up_b"]) @ w["down_w"].t() + w["down_b"]))
    return torch.stack(out)


def exact(case, seed):
    c = case
    if c["kind"] in ("block", "step"):
        s, x, cond, weights = _block_inputs(c, seed)
        x, cond = x.double(), cond.double()
        for w in weights:
            x = _exact_block(s, x, cond, w)
        return x
    if c["kind"] == "attention":
        q, k, vt = _attention_inputs(c, seed)
        B, H, L, d = c["batch"], c["heads"], c["keys"], c["head_dim"]
        o = torch.empty((B, c["q_count"], H, d), dtype=torch.float64, device=DEV)
        for b in range(B):
            for h in range(H):
                rows = q[b, h, c["q_begin"]:c["q_begin"] + c["q_count"]].double() * math.log(2)
                o[b, :, h] = _softmax_rows(rows, k[b, h, :L].double(), vt[b, h, :, :L].double().t().contiguous())
        return o.view(B * c["q_count"], H * d)
    if c["kind"] == "gemm":
        t = {n: v.double() for n, v in _gemm_inputs(c, seed).items()}
        u = t["a"] @ t["b"].t() + t["bias"]
        if c["epilogue"] == "gated":
            return t["resid"] + t["gate"] * u
        return _gelu(u) if c["epilogue"] == "gelu" else u
    x, w, bias = (t.double() for t in _vae_inputs(c, seed))
    H, Wd = c["h"], c["w"]
    r0, r1 = 2 * c["row_begin"], 2 * (c["row_begin"] + c["rows"])
    y = bias.expand(c["n"], r1 - r0, 2 * Wd, c["co"]).clone()
    for f in range(c["n"]):
        for ky in range(3):
            for kx in range(3):
                # output rows and columns whose tap (ky, kx) lies inside the upsampled image, and their source pixels
                u = torch.arange(max(r0, 1 - ky), min(r1, 2 * H + 1 - ky), device=DEV)
                v = torch.arange(max(0, 1 - kx), min(2 * Wd, 2 * Wd + 1 - kx), device=DEV)
                z = x[f] @ w[:, ky, kx].t().contiguous()
                y[f, u[0] - r0:u[-1] + 1 - r0, v[0]:v[-1] + 1] += z[(u + ky - 1) // 2][:, (v + kx - 1) // 2]
    return y
