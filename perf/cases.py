"""The work that a program has this library do, as cases that can be timed and checked.

A denoising iteration is dominated by transformer layers and the fused LM head, so most cases are one
layer (``dcl_debug_layer``: a decode loop's layer, on a given residual stream) or the head
(``dcl_score_hidden``), at the sizes the decode loop meets:

* few tokens: one sequence's block and its draft look-ahead over a cached prefix (prefix-KV decode);
* one whole short sequence (128-token prompt + 256 generated), one whole long one (256 + 1024);
* batches: eight cached decodes at once, four whole sequences of 768, three of an odd length;
* the head over one window, one generation region, a batch of regions.

The rest are whole calls: a denoising step (statistics of every scored row), a whole iteration of a
tiny model, where launches count (step and selection), and ``dcl_kv_append`` over a prompt (prefill).

Geometries are the LLaDA-8B and Dream-7B (GQA, biases) shapes and the two-layer tiny model. A layer
case carries a small vocabulary and a head case a small layer, which their calls never read: inputs
stay quick to make. Weights are N(0, 0.02^2) in bf16, as everywhere here.

``exact`` evaluates the same definition in float64 torch, with bfloat16 rounding exactly where the
library's documented storage points are (normalised operands, q/k/v, attention output, SwiGLU product).
"""
import math
from types import SimpleNamespace

import torch

import paper_2607_20467_amd as dcl

# the geometries of the models (rope base, eps: the published models' own)
MODELS = {
    "llada-8b": dict(d_model=4096, n_heads=32, n_kv_heads=32, head_dim=128, d_ffn=12288, vocab=126464,
                     rms_eps=1e-5, rope_base=5e5, qkv_bias=False),
    "dream-7b": dict(d_model=3584, n_heads=28, n_kv_heads=4, head_dim=128, d_ffn=18944, vocab=152064,
                     rms_eps=1e-6, rope_base=1e6, qkv_bias=True),
    "tiny": dict(d_model=256, n_heads=4, n_kv_heads=4, head_dim=64, d_ffn=688, vocab=4096,
                 rms_eps=1e-5, rope_base=1e4, qkv_bias=False),
}
# LM-head multiplier that spreads the top-1 confidences over (0, 1)
LM_SCALE = {"llada-8b": 6.0, "dream-7b": 6.5, "tiny": 20.0}
STD = 0.02
STATS = ("top1", "top2", "conf", "p2", "lse", "entropy")
# What a whole call through layers returns here. Its ids are left out (and with them the committed tokens):
# with random weights about one row in a hundred is a near-tie that float32 noise decides, so two correct
# implementations differ there; the head cases return ids, from given hidden states.
SMOOTH = ("conf", "p2", "lse", "entropy")
MAX_POSITIONS = 4096


def listed():
    return [
        # prefix-KV decode of one user: 32-token block + 32 drafts over a ragged cached prefix
        {"name": "layer llada 1x64 kv323", "op": "layer", "model": "llada-8b", "batch": 1, "seq": 64, "prefix": 323},
        # the headline step's layer: 128-token prompt + 256 generated positions
        {"name": "layer llada 1x384", "op": "layer", "model": "llada-8b", "batch": 1, "seq": 384, "prefix": 0},
        # eight cached decodes together, 1216-token prefixes
        {"name": "layer llada 8x64 kv1216", "op": "layer", "model": "llada-8b", "batch": 8, "seq": 64,
         "prefix": 1216},
        # three whole sequences of an odd length (GQA, biases)
        {"name": "layer dream 3x203", "op": "layer", "model": "dream-7b", "batch": 3, "seq": 203, "prefix": 0},
        # long generation: 256-token prompt + 1024 generated positions
        {"name": "layer llada 1x1280", "op": "layer", "model": "llada-8b", "batch": 1, "seq": 1280, "prefix": 0},
        # the largest batch of whole sequences: 4 x (256 + 512)
        {"name": "layer dream 4x768", "op": "layer", "model": "dream-7b", "batch": 4, "seq": 768, "prefix": 0},
        # scoring one 32-token window
        {"name": "head llada 32", "op": "head", "model": "llada-8b", "rows": 32},
        # scoring a 256-token generation region
        {"name": "head llada 256", "op": "head", "model": "llada-8b", "rows": 256},
        # scoring four regions of 480 open positions
        {"name": "head dream 1920", "op": "head", "model": "dream-7b", "rows": 1920},
        # one iteration (step + selection) of the tiny model: launch latency
        {"name": "iteration tiny 1x96", "op": "iteration", "model": "tiny", "layers": 2, "batch": 1, "seq": 96,
         "prompt": 32, "window": 16},
        # a whole step (embedding to statistics) of a two-layer slice, an odd length, mask id left out
        {"name": "step llada 1x329", "op": "step", "model": "llada-8b", "layers": 2, "batch": 1, "seq": 329,
         "prompt": 73, "suppress": True},
        # prefill: keys and values of a prompt into an empty cache, two-layer slice
        {"name": "append llada 1x730", "op": "append", "model": "llada-8b", "layers": 2, "batch": 1, "seq": 730,
         "prefix": 0, "capacity": 1024},
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(("layer", "layer", "layer", "layer", "head", "head", "append", "step", "iteration"))
    model = rng.choice(("llada-8b", "llada-8b", "dream-7b"))
    batch = rng.choice((1, 1, 1, 2, 3, 4, 8))
    if op == "head":
        return {"op": op, "model": model, "rows": _log(rng, 16, 1920)}
    if op == "iteration":
        seq = _log(rng, 48, 640)
        return {"op": op, "model": "tiny", "layers": 2, "batch": batch, "seq": seq, "prompt": seq // 3, "window": 16}
    if op == "step":
        seq = _log(rng, 96, 700)
        return {"op": op, "model": model, "layers": 2, "batch": 1, "seq": seq, "prompt": seq // 4,
                "suppress": rng.random() < 0.5}
    if op == "append":
        prefix = rng.choice((0, _log(rng, 64, 1500)))
        seq = _log(rng, 16, 512) if prefix else _log(rng, 64, 1280)
        return {"op": op, "model": model, "layers": 2, "batch": 1, "seq": seq, "prefix": prefix,
                "capacity": (prefix + seq + 263) // 8 * 8}
    if rng.random() < 0.5:  # cached decode: blocks and drafts over a prefix
        return {"op": op, "model": model, "batch": batch, "seq": _log(rng, 16, 192), "prefix": _log(rng, 64, 2048)}
    return {"op": op, "model": model, "batch": batch, "seq": _log(rng, 64, 2600 // batch), "prefix": 0}


# ---------------------------------------------------------------------------------------- inputs

def _geometry(case):
    g = dict(MODELS[case["model"]], n_layers=case.get("layers", 1))
    if case["op"] in ("layer", "append"):
        g["vocab"] = 2048                                     # the vocabulary is not what these calls use
    if case["op"] == "head":
        g.update(n_heads=1, n_kv_heads=1, head_dim=64, d_ffn=16)  # nor this call the layer
    return SimpleNamespace(mask_id=g["vocab"] - 1, **g)


def _weights(g, case, gen):
    """Tensors in dcl_load_weights' order, bf16 on the device."""
    d, hd, kd, F, V = g.d_model, g.n_heads * g.head_dim, g.n_kv_heads * g.head_dim, g.d_ffn, g.vocab

    def mat(*shape, std=STD):
        return torch.randn(shape, generator=gen, device="cuda").mul_(std).to(torch.bfloat16)

    def gain():
        return torch.randn(d, generator=gen, device="cuda").mul_(0.1).add_(1.0).to(torch.bfloat16)

    def bias(n):
        return mat(n) if g.qkv_bias else None

    out = [mat(V, d)]
    for _ in range(g.n_layers):
        out += [mat(hd, d), mat(kd, d), mat(kd, d), bias(hd), bias(kd), bias(kd), mat(d, hd), mat(F, d), mat(F, d),
                mat(d, F), gain(), gain()]
    out += [gain(), mat(V, d, std=STD * LM_SCALE[case["model"]])]
    return out


def _inputs(case, seed):
    """(geometry, weights, everything else the call takes), from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    g = _geometry(case)
    x = {"weights": _weights(g, case, gen)}
    op = case["op"]
    if op == "head":
        x["hidden"] = torch.randn((case["rows"], g.d_model), generator=gen, device="cuda").to(torch.bfloat16)
        return g, x
    B, S, P = case["batch"], case["seq"], case.get("prefix", 0)
    if op == "layer":
        x["r"] = torch.randn((B * S, g.d_model), generator=gen, device="cuda")
    else:
        x["tokens"] = torch.randint(0, g.vocab - 2, (B, S), generator=gen, device="cuda", dtype=torch.int32)
    if "prompt" in case:                                       # generation region: masked
        x["tokens"][:, case["prompt"]:] = g.mask_id
        x["p"] = torch.full((B,), case["prompt"], dtype=torch.int32, device="cuda")
    cap = case.get("capacity", (P + 7) // 8 * 8)
    if cap:
        def cache(*shape):
            return torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
        x["k"] = [cache(B, g.n_kv_heads, cap, g.head_dim) for _ in range(g.n_layers)]
        x["v"] = [cache(B, g.n_kv_heads, g.head_dim, cap) for _ in range(g.n_layers)]
        x["kv"] = (x["k"], x["v"], P, cap)
    return g, x


def prepare(case, seed):
    g, x = _inputs(case, seed)
    runner = dcl.Runner(g, x.pop("weights"), max_positions=MAX_POSITIONS)
    s = SimpleNamespace(case=case, g=g, runner=runner, kv=None, **{k: v for k, v in x.items() if k != "kv"})
    s.kv = x.get("kv")
    op = case["op"]
    if op == "head":
        s.ws_bytes = dcl.dcl_score_workspace_bytes(runner.model, case["rows"])
        s.ws = torch.empty(s.ws_bytes, dtype=torch.uint8, device="cuda")
        s.stats = {k: v.view(-1) for k, v in runner.new_stats(1, case["rows"]).items()}
        return s
    B, S, P = case["batch"], case["seq"], case.get("prefix", 0)
    s.ws, s.ws_bytes = runner.workspace(B, S, P)
    if op == "layer":
        s.taps = {"r_out": torch.empty_like(s.r)}
    elif op in ("step", "iteration"):
        s.stats = runner.new_stats(B, S)
        s.flags = dcl.DCL_SCORE_SUPPRESS_MASK if case.get("suppress") else 0
    if op == "iteration":
        s.tokens0, s.p0 = s.tokens.clone(), s.p.clone()
    return s


def run(s):
    op, c, m = s.case["op"], s.case, s.runner.model
    if op == "head":
        dcl.dcl_score_hidden(m, s.hidden, c["rows"], s.stats, s.ws, s.ws_bytes)
        return s.stats
    B, S = c["batch"], c["seq"]
    if op == "layer":
        dcl.dcl_debug_layer(m, B, S, s.kv, 0, s.r, s.taps, s.ws, s.ws_bytes)
        return s.taps["r_out"]
    if op == "append":
        dcl.dcl_kv_append(m, s.tokens, B, S, s.kv, s.ws, s.ws_bytes)
        return {"k": s.k, "v": s.v}
    if op == "step":
        dcl.dcl_denoise_step(m, s.tokens, B, S, s.p, S, s.kv, s.flags, s.stats, s.ws, s.ws_bytes)
        return {k: s.stats[k] for k in SMOOTH}
    # one iteration from the same state (selection updates tokens and p in place)
    s.tokens.copy_(s.tokens0)
    s.p.copy_(s.p0)
    dcl.dcl_denoise_step(m, s.tokens, B, S, s.p, S, s.kv, s.flags, s.stats, s.ws, s.ws_bytes)
    dcl.dcl_select_contiguous(s.tokens, B, S, s.p, S, c["window"], 0.7, 0.98, s.g.mask_id, s.stats)
    return {k: s.stats[k] for k in SMOOTH}


# ---------------------------------------------------------------------------------------- what a pass needs

def work(case):
    g, op = _geometry(case), case["op"]
    d, F, V = g.d_model, g.d_ffn, g.vocab
    hd, kd = g.n_heads * g.head_dim, g.n_kv_heads * g.head_dim
    if op == "head":
        R = case["rows"]
        return {"bytes": 2 * V * d + 2 * R * d + 24 * R, "flops": 2 * R * V * d}
    B, S, P, L = case["batch"], case["seq"], case.get("prefix", 0), case.get("layers", 1)
    T = B * S
    qkv, rest = (hd + 2 * kd) * d, hd * d + 3 * F * d
    attn = 4 * T * hd * (P + S)
    cache = 2 * B * P * kd * 2
    if op == "layer":
        return {"bytes": 2 * (qkv + rest) + cache + 8 * T * d, "flops": 2 * T * (qkv + rest) + attn}
    if op == "append":  # the last layer ends with its keys and values
        kv_rows = 2 * kd * d
        return {"bytes": 2 * (L - 1) * (qkv + rest) + 2 * kv_rows + (L - 1) * cache + 2 * T * d + 4 * T * kd * L,
                "flops": (L - 1) * (2 * T * (qkv + rest) + attn) + 2 * T * kv_rows}
    R = B * (S - case["prompt"])
    return {"bytes": 2 * L * (qkv + rest) + 2 * V * d + 2 * T * d + 24 * T,
            "flops": L * (2 * T * (qkv + rest) + attn) + 2 * R * V * d}


def tolerance(case):
    # About four times the error against exact() that two correct float32 orders both show. On given bf16
    # hidden states that is float32 noise (2e-5). Through a layer, a value within float32 noise of a bf16
    # rounding boundary rounds the other way, and each further storage point amplifies it: after one layer
    # the float32 residual is off by 1.7e-3, the next layer's bf16 keys by 3.7e-3, and the statistics by
    # that times the logits' spread.
    if case["op"] == "head":
        return {"rel": 1e-4, "max": 1e-3, "differ": 0.01}
    if case["op"] == "layer":
        return {"rel": 7e-3, "max": 0.1}
    if case["op"] == "append":
        return {"rel": 1.5e-2, "max": 0.2}
    return {"rel": 3e-2, "max": 0.7}


# ---------------------------------------------------------------------------------------- float64 torch

def _bf(x):
    return x.to(torch.float32).to(torch.bfloat16).to(torch.float64)


def _norm(r, gain, eps):
    return _bf(r * torch.rsqrt(r.square().mean(-1, keepdim=True) + eps) * gain.double())


def _rope(x, pos, base):
    half = x.shape[-1] // 2
    inv = base ** (-torch.arange(half, device="cuda", dtype=torch.float64) * 2.0 / x.shape[-1])
    ang = pos.double()[:, None] * inv                          # [S, half]
    c, s = ang.cos()[:, None, :], ang.sin()[:, None, :]        # heads broadcast
    a, b = x[..., :half], x[..., half:]
    return torch.cat((a * c - b * s, b * c + a * s), -1)


def _layer(g, w, r, B, S, P, cache):
    """One layer on r [B*S, d] (float64); returns (r_out, k [B, Hkv, S, dh], v [B, Hkv, S, dh])."""
    wq, wk, wv, bq, bk, bv, wo, wg, wu, wd, g1, g2 = w
    H, Hk, dh = g.n_heads, g.n_kv_heads, g.head_dim
    u = _norm(r, g1, g.rms_eps)

    def proj(m, b, heads):
        y = u @ m.double().t()
        return (y + b.double() if b is not None else y).view(B, S, heads, dh)
    pos = P + torch.arange(S, device="cuda")
    q = _bf(torch.stack([_rope(x, pos, g.rope_base) for x in proj(wq, bq, H)]))
    k = _bf(torch.stack([_rope(x, pos, g.rope_base) for x in proj(wk, bk, Hk)])).transpose(1, 2)
    v = _bf(proj(wv, bv, Hk)).transpose(1, 2)
    o = torch.empty((B, S, H, dh), dtype=torch.float64, device="cuda")
    for b in range(B):
        for h in range(H):
            n = h // (H // Hk)
            kk, vv = k[b, n], v[b, n]
            if P:
                kk = torch.cat((cache[0][b, n, :P].double(), kk))
                vv = torch.cat((cache[1][b, n, :, :P].double().t(), vv))
            prob = torch.softmax(q[b, :, h] @ kk.t() / math.sqrt(dh), -1)
            o[b, :, h] = prob @ vv
    r = r + _bf(o).view(B * S, H * dh) @ wo.double().t()
    u2 = _norm(r, g2, g.rms_eps)
    a = _bf(torch.nn.functional.silu(u2 @ wg.double().t()) * (u2 @ wu.double().t()))
    return r + a @ wd.double().t(), k, v


def _row_stats(hidden, lm, exclude):
    """conf, p2, lse, entropy of float64 hidden rows, the vocabulary's logits in float64."""
    out = {k: torch.empty(hidden.shape[0], dtype=torch.float64, device="cuda") for k in ("conf", "p2", "lse", "entropy")}
    w = lm.double()
    for i in range(0, hidden.shape[0], 512):
        logits = hidden[i:i + 512] @ w.t()
        if exclude is not None:
            logits[:, exclude] = -math.inf
        lse = logits.logsumexp(-1)
        top = logits.topk(2, -1).values
        prob = torch.softmax(logits, -1)
        out["conf"][i:i + 512], out["p2"][i:i + 512] = torch.exp(top - lse[:, None]).unbind(-1)
        out["lse"][i:i + 512] = lse
        out["entropy"][i:i + 512] = lse - (prob * logits.masked_fill(prob == 0, 0.0)).sum(-1)
    return out


def exact(case, seed):
    g, x = _inputs(case, seed)
    w, op = x["weights"], case["op"]
    layer = lambda l: w[1 + 12 * l:13 + 12 * l]  # noqa: E731
    if op == "head":
        return {**dict.fromkeys(STATS), **_row_stats(x["hidden"].double(), w[-1], None)}
    B, S, P = case["batch"], case["seq"], case.get("prefix", 0)
    if op == "layer":
        return _layer(g, layer(0), x["r"].double(), B, S, P, (x["k"][0], x["v"][0]) if P else None)[0]
    r = w[0].double()[x["tokens"].long()].view(B * S, g.d_model)
    for l in range(g.n_layers):
        r, k, v = _layer(g, layer(l), r, B, S, P, (x["k"][l], x["v"][l]) if P else None)
        if op == "append":
            x["k"][l], x["v"][l] = x["k"][l].double(), x["v"][l].double()
            x["k"][l][:, :, P:P + S] = k
            x["v"][l][:, :, :, P:P + S] = v.transpose(2, 3)
    if op == "append":
        return {"k": x["k"], "v": x["v"]}
    full = {"conf": -1.0, "p2": -1.0, "lse": 0.0, "entropy": -1.0}
    full = {k: torch.full((B, S), v, dtype=torch.float64, device="cuda") for k, v in full.items()}
    hidden = _norm(r, w[-2], g.rms_eps).view(B, S, -1)[:, case["prompt"]:]
    got = _row_stats(hidden.reshape(-1, g.d_model), w[-1], g.mask_id if case.get("suppress") else None)
    for k, v in got.items():
        full[k][:, case["prompt"]:] = v.view(B, -1)
    return full
