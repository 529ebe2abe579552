"""The work this framework is used for, as measurable cases.

A case is one call sequence through the package's entry points on the shapes
of its configurations (ld_inputs.SHAPES and the benchmark):

  step    ld_stack_step: masks, forward and backward of a stack (a training
          step without the optimizer)
  fwd     ld_layer_fwd of one layer (training form, one mask draw)
  bwd     ld_layer_bwd of one layer whose forward ran before
  train   ld_layer_fwd then ld_layer_bwd of one layer
  eval    ld_stack_eval over a prompt, writing the key/value caches (prefill)
  decode  ld_stack_decode of n_new rows per sequence over those caches: one
          row is a token of plain decoding (or of a draft, with a layer
          subset), several rows the verify step of speculative decoding
  attn    ld_attn_fwd then ld_attn_bwd_noalloc, attention on its own

The masks' seed and step belong to the case, so which sequences a layer keeps
is the same for every input seed; hidden states, weights, upstream gradients
and caches come from the input seed.  Hidden states are N(0, 1), weights
N(0, 0.02), gains 1 + N(0, 0.02), caches N(0, 0.9) (what N(0, 0.02)
projections of unit-RMS rows of d = 2048 give).

Calls that work in place start from a copy of their input (the embedding's
output, the loss gradient), made on the stream as part of the pass.
"""
import math

import numpy as np
import torch

import paper_2609_05275_amd as ld

DEV = "cuda:0"
KEYS = ("g_attn", "w_qkv", "w_o", "g_mlp", "w_gate_up", "w_down")


# ------------------------------------------------------------------- cases

def _case(name, kind, layers, d, heads, f, seq, batch, **kw):
    c = dict(name=name, kind=kind, layers=layers, d=d, heads=heads, f=f, seq=seq, batch=batch, dtype="bf16",
             block=0, gran=0, p_max=0.2, first=0, depth=layers, mask_seed=0, step=1000, pos=0, n_new=0,
             s_max=0, every=1)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: the tiny float32 stack (parity runs, debugging on
        # small models), where launches and host time are everything
        _case("step_tiny_f32", "step", 2, 64, 4, 172, 32, 8, dtype="f32"),
        # interactive decoding: one sequence, one token through the whole
        # 1B-shape model over an odd cache length
        _case("decode_1b_b1", "decode", 16, 2048, 16, 5504, 64, 1, pos=777, n_new=1, s_max=1024),
        # batched drafting: one token per sequence, every other layer active,
        # over full caches
        _case("draft_1b_b8", "decode", 16, 2048, 16, 5504, 64, 8, pos=2047, n_new=1, s_max=2056, every=2),
        # the verify step after a draft of 5: six rows per sequence through
        # every layer
        _case("verify_1b_b8", "decode", 16, 2048, 16, 5504, 64, 8, pos=1500, n_new=6, s_max=1536),
        # prefill of three ragged prompts with an early exit after 12 layers
        _case("prefill_1b", "eval", 12, 2048, 16, 5504, 1088, 3, s_max=1152),
        # one 1B-shape layer of a training step, forward and backward apart
        # (rate of a middle layer: 7 of the 8 sequences kept)
        _case("fwd_1b", "fwd", 1, 2048, 16, 5504, 2048, 8, first=8, depth=16),
        _case("bwd_1b", "bwd", 1, 2048, 16, 5504, 2048, 8, first=8, depth=16),
        # the paper's own block (ALiBi, squared ReLU) at its 3.9B
        # architecture, a deep layer on a ragged batch
        _case("train_3p9b", "train", 1, 2048, 16, 16384, 1472, 5, block=1, first=30, depth=40),
        # a 7B-shape layer at its full sequence length
        _case("train_7b", "train", 1, 4096, 32, 11008, 4096, 4, first=16, depth=32),
        # the 125M-shape training step, whole: small GEMMs, 64-wide heads
        _case("step_125m", "step", 12, 768, 12, 2048, 1024, 8),
        # the 1B-shape training step, whole (the benchmark's workload)
        _case("step_1b", "step", 16, 2048, 16, 5504, 2048, 8),
        # attention on its own, 64-wide heads, ragged length, both directions
        _case("attn_d64", "attn", 1, 1536, 24, 4096, 1984, 3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _train_flops(c):
    fw = (3 if c["block"] == 0 else 2) * c["d"] * c["f"]
    t = c["batch"] * c["seq"]
    return 3 * c["layers"] * (2 * t * (4 * c["d"] ** 2 + fw) + 2 * t * c["d"] * (c["seq"] + 1))


def draw(rng):
    """One more case of the same kinds and ranges."""
    kind = rng.choice(["step", "step_f32", "fwd", "bwd", "train", "eval", "decode", "decode", "verify", "attn"])
    if kind == "step_f32":
        dh = rng.choice([16, 32, 64])
        heads = rng.randint(2, 6)
        d = dh * heads
        c = _case("", "step", rng.randint(1, 4), d, heads, 4 * rng.randint(d // 4, 3 * d // 4),
                  rng.randint(17, 128), rng.randint(1, 12), dtype="f32", block=rng.randint(0, 1))
    else:
        dh = rng.choice([64, 128, 128])
        heads = rng.choice([8, 12, 16, 20, 24, 32])
        d = dh * heads
        block = rng.choice([0, 0, 1])
        unit = rng.choice([8, 128])
        f = unit * _log_int(rng, d * 2 // unit, d * (3 if block == 0 else 8) // unit)
        if kind in ("decode", "verify"):
            batch = _log_int(rng, 1, 16)
            n_new = 1 if kind == "decode" else rng.randint(2, 8)
            pos = _log_int(rng, 30, 4000)
            c = _case("", "decode", rng.randint(2, 8), d, heads, f, 64, batch, block=block, pos=pos, n_new=n_new,
                      s_max=pos + n_new + rng.randint(0, 200), every=rng.choice([1, 1, 2]))
        elif kind == "attn":
            seq = 64 * _log_int(rng, 2, 64)
            batch = max(1, min(rng.randint(1, 8), 2 ** 21 // (heads * seq)))
            c = _case("", "attn", 1, d, heads, f, seq, batch, block=block)
        else:
            c = _case("", kind, rng.randint(2, 6) if kind in ("step", "eval") else 1, d, heads, f,
                      64 * _log_int(rng, 2, 64), _log_int(rng, 1, 32), block=block)
            if kind == "eval":
                c["s_max"] = c["seq"] + rng.randint(0, 128)
            else:
                c["p_max"] = rng.choice([0.0, 0.1, 0.2, 0.5, 0.8])
                c["gran"] = rng.choice([0, 0, 1, 2, 3])
                if kind != "step":
                    c["depth"] = rng.randint(2, 32)
                    c["first"] = rng.randrange(c["depth"])
            # no more than the 1B-shape step's work and memory
            while _train_flops(c) > 8.0e13 or c["layers"] * c["batch"] * c["seq"] > 16 * 16384:
                if c["batch"] > 1:
                    c["batch"] //= 2
                else:
                    c["seq"] = max(64, c["seq"] // 128 * 64)
    c["mask_seed"], c["step"] = rng.randrange(1 << 30), rng.randrange(100000)
    del c["name"]
    return c


# ------------------------------------------------------------ masks, sizes

def _rates(c):
    """ILD depth distribution at the end of its ramp: p_max l / (depth - 1)."""
    den = max(1, c["depth"] - 1)
    return [float(np.float32(c["p_max"] * (c["first"] + l) / den)) for l in range(c["layers"])]


def _word(b, layer, step, per_batch, seed, m):
    """Word m of Philox4x64-10 block (b, layer, step, per_batch), from numpy's
    generator (which increments its counter before the first block)."""
    ctr = b | (layer << 64) | (step << 128) | (per_batch << 192)
    ctr = (ctr - 1) % (1 << 256)
    words = [(ctr >> (64 * i)) & (2 ** 64 - 1) for i in range(4)]
    g = np.random.Philox(counter=np.array(words, dtype=np.uint64), key=np.array([seed, 0], dtype=np.uint64))
    return int(g.random_raw(4)[m])


def _kept(c):
    """Per layer the kept samples of the attention and FFN masks, and r."""
    out = []
    per_batch = 1 if c["gran"] & 2 else 0
    for l, p in enumerate(_rates(c)):
        thr = int(np.float64(np.float32(p)) * 2.0 ** 64)

        def keep(m):
            if p >= 1:
                return []
            if p <= 0:
                return list(range(c["batch"]))
            return [b for b in range(c["batch"])
                    if _word(0 if per_batch else b, c["first"] + l, c["step"], per_batch, c["mask_seed"], m) >= thr]
        a = keep(0)
        out.append((a, keep(1) if c["gran"] & 1 else a, 0.0 if p >= 1 else float(np.float32(1.0 / (1.0 - p)))))
    return out


def _active(c):
    return [l % c["every"] == 0 for l in range(c["layers"])]


def _weight_shapes(c):
    d, f = c["d"], c["f"]
    return dict(g_attn=(d,), w_qkv=(3 * d, d), w_o=(d, d), g_mlp=(d,),
                w_gate_up=((2 if c["block"] == 0 else 1) * f, d), w_down=(d, f))


def work(case):
    """Weights and inputs once in, outputs once out; a saved context or a
    workspace is the implementation's own."""
    c = case
    d, f, S, B, L = c["d"], c["f"], c["seq"], c["batch"], c["layers"]
    es = 4 if c["dtype"] == "f32" else 2
    n_ffn = 3 if c["block"] == 0 else 2
    w_attn, w_ffn = 4 * d * d, n_ffn * d * f
    n_w = w_attn + w_ffn + 2 * d
    dh_pairs = 2 * d * S * (S + 1)        # causal QK^T and PV of one sequence
    if c["kind"] == "attn":
        # forward: qkv in, o and lse out; backward: qkv, o, go, lse in, gqkv out
        t = B * S
        return dict(bytes=float(es * t * d * (3 + 1 + 3 + 1 + 1 + 3) + 8 * B * c["heads"] * S),
                    flops=3.0 * B * dh_pairs)
    if c["kind"] == "decode":
        n, keys = c["n_new"], c["pos"] + c["n_new"]
        la = sum(_active(c))
        flops = la * B * n * (2.0 * (w_attn + w_ffn) + 4.0 * d * keys)
        return dict(bytes=float(la * (2 * n_w + 2 * B * keys * 2 * d) + 4 * B * n * d), flops=flops)
    if c["kind"] == "eval":
        flops = L * B * (2.0 * S * (w_attn + w_ffn) + dh_pairs)
        return dict(bytes=float(L * (2 * n_w + 2 * B * S * 2 * d) + 4 * B * S * d), flops=flops)
    fwd = kept = 0.0
    for a, m, _ in _kept(c):
        fwd += len(a) * (2.0 * S * w_attn + dh_pairs) + len(m) * 2.0 * S * w_ffn
        kept += max(len(a), len(m))
    x_io = 2.0 * es * S * d * kept         # kept rows in and out
    if c["kind"] == "fwd":
        return dict(bytes=L * es * n_w + x_io, flops=fwd)
    bwd_bytes = L * (es + 4.0) * n_w + x_io
    if c["kind"] == "bwd":                 # the saved activations come in too
        per_tok = es * (d + 3 * d + d + d + (n_ffn - 1) * f + f) + 8 * d
        return dict(bytes=bwd_bytes + kept * S * per_tok, flops=2.0 * fwd)
    return dict(bytes=bwd_bytes + L * es * n_w + x_io, flops=3.0 * fwd)


def tolerance(case):
    """About four times the distance from the 64-bit values measured for one
    layer (bf16 operands, float32 sums): 0.2 % in the forward, 0.3-0.8 % in
    gradients.  A whole stack of bf16 decoding or evaluation layers, whose
    residual stream is bf16, is 1-1.8 % away, so another implementation of it
    is up to 1.5 times that from this one.  float32: 4e-7."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    if case["kind"] in ("attn", "fwd"):
        return {"rel": 1e-2, "max": 0.25}
    return {"rel": 3e-2, "max": 0.5}


# ------------------------------------------------------------------ inputs

def _gen(seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1_000_003 + tag) & 0x7FFFFFFFFFFFFFFF)
    return g


def _normal(shape, seed, tag, scale, dtype, mean=0.0):
    t = torch.randn(shape, generator=_gen(seed, tag), device=DEV, dtype=torch.float32)
    return t.mul_(scale).add_(mean).to(dtype)


def _dt(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _weights(c, seed, l):
    return {k: _normal(s, seed, 100 * l + i, 0.02, _dt(c), mean=1.0 if len(s) == 1 else 0.0)
            for i, (k, s) in enumerate(_weight_shapes(c).items())}


def _hidden(c, seed, tag, rows=None):
    return _normal((c["batch"], c["seq"] if rows is None else rows, c["d"]), seed, tag, 1.0, _dt(c))


def _cache(c, seed, l):
    return _normal((c["batch"], c["s_max"], 2 * c["d"]), seed, 60000 + l, 0.9, torch.bfloat16)


_X, _DX, _QKV, _GO = 50001, 50002, 50003, 50004


def prepare(case, seed):
    c = case
    B, S, L, dh = c["batch"], c["seq"], c["layers"], c["d"] // c["heads"]
    if c["kind"] == "attn":
        n = B * S
        return dict(c=c, qkv=_normal((n, 3 * c["d"]), seed, _QKV, 0.9, _dt(c)), go=_normal((n, c["d"]), seed, _GO, 1.0, _dt(c)),
                    o=torch.empty(n, c["d"], dtype=_dt(c), device=DEV),
                    lse=torch.empty(B, c["heads"], S, dtype=torch.float32, device=DEV),
                    gqkv=torch.empty(n, 3 * c["d"], dtype=_dt(c), device=DEV), dh=dh)
    cfg = ld.config(B, S, c["d"], c["heads"], c["f"], ld.LD_F32 if c["dtype"] == "f32" else ld.LD_BF16,
                    block_kind=c["block"], granularity=c["gran"])
    w = [_weights(c, seed, l) for l in range(L)]

    def buf(n):
        return torch.empty(n, dtype=torch.uint8, device=DEV)
    s = dict(c=c, cfg=cfg, w=w, p=_rates(c))
    if c["kind"] == "decode":
        s["x0"] = _hidden(c, seed, _X, c["n_new"])
        s["active"] = _active(c)
        s["kv"] = [_cache(c, seed, l) if a else None for l, a in enumerate(s["active"])]
        s["ws"] = buf(ld.ld_decode_ws_bytes(cfg, c["n_new"], c["s_max"]))
        s["x"] = torch.empty_like(s["x0"])
        return s
    s["x0"] = _hidden(c, seed, _X)
    s["x"] = torch.empty_like(s["x0"])
    if c["kind"] == "eval":
        s["kv"] = [torch.zeros(B, c["s_max"], 2 * c["d"], dtype=torch.bfloat16, device=DEV) for _ in range(L)]
        s["ws"] = buf(ld.ld_eval_ws_bytes(cfg))
        return s
    if c["kind"] != "fwd":
        s["dx0"] = _hidden(c, seed, _DX)
        s["dx"] = torch.empty_like(s["dx0"])
        # gradients of a parameter stacked over the layers, as an optimizer keeps them
        s["grads"] = {k: torch.empty((L,) + v, dtype=torch.float32, device=DEV) for k, v in _weight_shapes(c).items()}
        s["dw"] = [{k: g[l] for k, g in s["grads"].items()} for l in range(L)]
    if c["kind"] == "step":
        s["ws"] = buf(ld.ld_stack_ws_bytes(cfg, L))
    else:
        s["ctx"] = buf(ld.ld_layer_ctx_bytes(cfg))
        s["ws"] = buf(ld.ld_layer_ws_bytes(cfg))
    if c["kind"] == "bwd":
        s["x"].copy_(s["x0"])
        _layer_fwd(s)
    return s


def _layer_fwd(s):
    c = s["c"]
    ld.ld_layer_fwd(s["cfg"], s["w"][0], c["first"], s["p"][0], c["mask_seed"], c["step"], s["x"], s["ctx"], s["ws"])


def run(state):
    s = state
    c = s["c"]
    kind = c["kind"]
    if kind == "attn":
        ld.ld_attn_fwd(c["batch"], c["seq"], c["heads"], s["dh"], s["qkv"], s["o"], s["lse"], alibi=c["block"])
        ld.ld_attn_bwd_noalloc(c["batch"], c["seq"], c["heads"], s["dh"], s["qkv"], s["o"], s["lse"], s["go"], s["gqkv"],
                               alibi=c["block"])
        return [s["o"], s["lse"], s["gqkv"]]
    if kind == "decode":
        s["x"].copy_(s["x0"])
        ld.ld_stack_decode(s["cfg"], s["w"], s["x"], s["kv"], c["s_max"], c["pos"], c["n_new"], s["ws"],
                           active=s["active"])
        return [s["x"], [k for k in s["kv"] if k is not None]]
    if kind == "eval":
        s["x"].copy_(s["x0"])
        ld.ld_stack_eval(s["cfg"], s["w"], s["x"], s["ws"], kv=s["kv"], s_max=c["s_max"])
        return [s["x"], s["kv"]]
    if kind == "fwd":
        s["x"].copy_(s["x0"])
        _layer_fwd(s)
        return [s["x"]]
    s["dx"].copy_(s["dx0"])
    if kind == "bwd":
        ld.ld_layer_bwd(s["cfg"], s["w"][0], s["ctx"], s["dx"], s["dw"][0], s["ws"])
        return [s["dx"], s["grads"]]
    s["x"].copy_(s["x0"])
    if kind == "train":
        _layer_fwd(s)
        ld.ld_layer_bwd(s["cfg"], s["w"][0], s["ctx"], s["dx"], s["dw"][0], s["ws"])
    else:
        ld.ld_stack_step(s["cfg"], s["w"], s["p"], c["mask_seed"], c["step"], s["x"], s["dx"], s["dw"], s["ws"])
    return [s["x"], s["dx"], s["grads"]]


# ---------------------------------------------------- the same in 64 bits

_F = torch.float64


def _slope(h, n_heads):
    n = 1
    while 2 * n <= n_heads:
        n *= 2
    return 2.0 ** (-8.0 * (h + 1) / n) if h < n else 2.0 ** (-4.0 * (2 * (h - n) + 1) / n)


def _scores(q, k, q0, slope):
    """Biased, scaled, causal scores of queries at positions q0.. over keys."""
    n, m = q.shape[0], k.shape[0]
    s = (q @ k.t().contiguous()) / math.sqrt(q.shape[1])
    i = torch.arange(q0, q0 + n, device=q.device)[:, None]
    j = torch.arange(m, device=q.device)[None, :]
    if slope:
        s -= slope * (i - j).to(_F)
    return s.masked_fill_(j > i, -math.inf)


def _attn_rows(q, k, v, q0, heads, alibi):
    """o and log-sum-exp; q [n, d], k, v [m, d]."""
    dh = q.shape[1] // heads
    o, lse = torch.empty_like(q), torch.empty(heads, q.shape[0], dtype=_F, device=q.device)
    for h in range(heads):
        c = slice(h * dh, (h + 1) * dh)
        s = _scores(q[:, c].contiguous(), k[:, c].contiguous(), q0, _slope(h, heads) if alibi else 0.0)
        lse[h] = torch.logsumexp(s, 1)
        o[:, c] = torch.exp(s - lse[h][:, None]) @ v[:, c].contiguous()
    return o, lse


def _attn_grad(qkv, o, lse, go, heads, alibi):
    d = o.shape[1]
    dh = d // heads
    g = torch.empty_like(qkv)
    for h in range(heads):
        q, k, v = (qkv[:, i * d + h * dh:i * d + (h + 1) * dh].contiguous() for i in range(3))
        c = slice(h * dh, (h + 1) * dh)
        p = torch.exp(_scores(q, k, 0, _slope(h, heads) if alibi else 0.0) - lse[h][:, None])
        goh = go[:, c].contiguous()
        ds = p * (goh @ v.t().contiguous() - (goh * o[:, c]).sum(1, keepdim=True)) / math.sqrt(dh)
        g[:, h * dh:(h + 1) * dh] = ds @ k
        g[:, d + h * dh:d + (h + 1) * dh] = ds.t().contiguous() @ q
        g[:, 2 * d + h * dh:2 * d + (h + 1) * dh] = p.t().contiguous() @ goh
    return g


def _rms(x, g):
    rstd = torch.rsqrt((x * x).mean(1, keepdim=True) + 1e-5)
    return x * rstd * g, rstd


def _rms_grad(x, rstd, g, gy):
    dg = (gy * x * rstd).sum(0)
    t = g * gy
    return rstd * t - x * rstd ** 3 * (x * t).mean(1, keepdim=True), dg


def _attn_block(c, w, x, r):
    h, rstd = _rms(x, w["g_attn"])
    qkv = h @ w["w_qkv"].t()
    d = c["d"]
    o, lse = _attn_rows(qkv[:, :d], qkv[:, d:2 * d], qkv[:, 2 * d:], 0, c["heads"], c["block"])
    return x + r * (o @ w["w_o"].t()), (h, rstd, qkv, o, lse)


def _ffn_act(c, uv):
    if c["block"]:
        return torch.clamp(uv, min=0) ** 2
    u, v = uv[:, :c["f"]], uv[:, c["f"]:]
    return u * torch.sigmoid(u) * v


def _ffn_block(c, w, z, r):
    h, rstd = _rms(z, w["g_mlp"])
    uv = h @ w["w_gate_up"].t()
    s = _ffn_act(c, uv)
    return z + r * (s @ w["w_down"].t()), (h, rstd, uv, s)


def _ffn_grad(c, w, z, r, gy, dw):
    _, (h, rstd, uv, s) = _ffn_block(c, w, z, r)
    gk = r * gy
    dw["w_down"] += gk.t() @ s
    gs = gk @ w["w_down"]
    if c["block"]:
        guv = gs * 2 * torch.clamp(uv, min=0)
    else:
        u, v = uv[:, :c["f"]], uv[:, c["f"]:]
        sg = torch.sigmoid(u)
        guv = torch.cat([gs * v * sg * (1 + u * (1 - sg)), gs * u * sg], 1)
    dw["w_gate_up"] += guv.t() @ h
    gx, dg = _rms_grad(z, rstd, w["g_mlp"], guv @ w["w_gate_up"])
    dw["g_mlp"] += dg
    return gy + gx


def _attn_block_grad(c, w, x, r, gz, dw):
    _, (h, rstd, qkv, o, lse) = _attn_block(c, w, x, r)
    gk = r * gz
    dw["w_o"] += gk.t() @ o
    gqkv = _attn_grad(qkv, o, lse, gk @ w["w_o"], c["heads"], c["block"])
    dw["w_qkv"] += gqkv.t() @ h
    gx, dg = _rms_grad(x, rstd, w["g_attn"], gqkv @ w["w_qkv"])
    dw["g_attn"] += dg
    return gz + gx


def _exact_train(c, seed):
    x = _hidden(c, seed, _X).to(_F)
    kept = _kept(c)
    xs, zs = [], []
    for l, (ka, kf, r) in enumerate(kept):
        w = {k: v.to(_F) for k, v in _weights(c, seed, l).items()}
        xs.append(x)
        z = x.clone()
        for b in ka:
            z[b] = _attn_block(c, w, x[b], r)[0]
        zs.append(z)
        x = z.clone()
        for b in kf:
            x[b] = _ffn_block(c, w, z[b], r)[0]
    if c["kind"] == "fwd":
        return [x]
    g = _hidden(c, seed, _DX).to(_F)
    dws = [None] * c["layers"]
    for l in range(c["layers"] - 1, -1, -1):
        ka, kf, r = kept[l]
        w = {k: v.to(_F) for k, v in _weights(c, seed, l).items()}
        dw = {k: torch.zeros(s, dtype=_F, device=DEV) for k, s in _weight_shapes(c).items()}
        for b in kf:
            g[b] = _ffn_grad(c, w, zs[l][b], r, g[b], dw)
        for b in ka:
            g[b] = _attn_block_grad(c, w, xs[l][b], r, g[b], dw)
        xs[l] = zs[l] = None
        dws[l] = dw
    grads = {k: torch.stack([dw[k] for dw in dws]) for k in KEYS}
    return [g, grads] if c["kind"] == "bwd" else [x, g, grads]


def _exact_decode(c, seed):
    n, d = c["n_new"], c["d"]
    x = _hidden(c, seed, _X, n).to(_F)
    kv = []
    for l, a in enumerate(_active(c)):
        if not a:
            continue
        w = {k: v.to(_F) for k, v in _weights(c, seed, l).items()}
        cache = _cache(c, seed, l).to(_F)
        h, _ = _rms(x.reshape(-1, d), w["g_attn"])
        qkv = (h @ w["w_qkv"].t()).reshape(c["batch"], n, 3 * d)
        cache[:, c["pos"]:c["pos"] + n] = qkv[:, :, d:]
        m = c["pos"] + n
        o = torch.stack([_attn_rows(qkv[b, :, :d], cache[b, :m, :d], cache[b, :m, d:], c["pos"], c["heads"],
                                    c["block"])[0] for b in range(c["batch"])])
        z = x.reshape(-1, d) + o.reshape(-1, d) @ w["w_o"].t()
        x = _ffn_block(c, w, z, 1.0)[0].reshape(c["batch"], n, d)
        kv.append(cache)
    return [x, kv]


def exact(case, seed):
    c = case
    if c["kind"] == "decode":
        return _exact_decode(c, seed)
    if c["kind"] == "attn":
        d, S, H = c["d"], c["seq"], c["heads"]
        qkv = _normal((c["batch"] * S, 3 * d), seed, _QKV, 0.9, _dt(c)).to(_F)
        go = _normal((c["batch"] * S, d), seed, _GO, 1.0, _dt(c)).to(_F)
        o, lse, g = torch.empty_like(go), torch.empty(c["batch"], H, S, dtype=_F, device=DEV), torch.empty_like(qkv)
        for b in range(c["batch"]):
            t = slice(b * S, (b + 1) * S)
            o[t], lse[b] = _attn_rows(qkv[t, :d], qkv[t, d:2 * d], qkv[t, 2 * d:], 0, H, c["block"])
            g[t] = _attn_grad(qkv[t], o[t], lse[b], go[t], H, c["block"])
        return [o, lse, g]
    if c["kind"] == "eval":
        x = _hidden(c, seed, _X).to(_F)
        kv = []
        for l in range(c["layers"]):
            w = {k: v.to(_F) for k, v in _weights(c, seed, l).items()}
            cache = torch.zeros(c["batch"], c["s_max"], 2 * c["d"], dtype=_F, device=DEV)
            x = x.clone()
            for b in range(c["batch"]):
                z, (_, _, qkv, _, _) = _attn_block(c, w, x[b], 1.0)
                cache[b, :c["seq"]] = qkv[:, c["d"]:]
                x[b] = _ffn_block(c, w, z, 1.0)[0]
            kv.append(cache)
        return [x, kv]
    return _exact_train(c, seed)
