"""Every GEMM tile configuration at the edges of its tiles: token counts one past or short of a tile, partly
filled fragment columns, weight rows that leave partial tiles, short K ranges and K splits, against float64.

Layers: dcl_debug_layer without RoPE (the projections are then plain products), each stage fed the GPU's own
input. A sum of K products in any order, every addition rounded, errs by at most (K + c) 2^-23 sum |terms|
(2^-23: twice the round-to-nearest unit, so truncating accumulators are covered); a bfloat16 store adds half
an ulp, at most 2^-8 of the value. Head: dcl_score_hidden on given rows, at the exact-input bar of the suite.
"""
import dataclasses

import pytest

import synth
from helpers import CONF_TOL, LOGIT_TOL, TIE_GAP

# (d_model, d_ffn, heads x 64, tokens): the plans of their four GEMMs cover every configuration (checked below)
LAYERS = [(384, 6144, 4, 17), (384, 6144, 4, 129), (384, 6144, 4, 200), (384, 6144, 4, 385), (384, 6144, 4, 449),
          (384, 6144, 4, 513), (384, 6144, 4, 700), (384, 6144, 4, 770), (384, 6144, 4, 1025), (384, 6144, 16, 1300),
          (1152, 3072, 2, 775), (1024, 3072, 2, 1361), (2048, 3072, 4, 705), (2048, 3072, 4, 768),
          (256, 3072, 4, 700), (1024, 3072, 16, 1025), (1024, 3072, 16, 600), (2048, 3072, 16, 1025),
          (1152, 12288, 2, 497), (400, 208, 4, 131),
          # one token tile (32 x 32 tiles; 32, 48 and 96 rows x 64 tokens): remainders of rows and tokens, short K
          (128, 6144, 4, 33), (128, 4160, 4, 63), (128, 8000, 4, 64), (128, 8320, 4, 64), (256, 2000, 4, 31), (1408, 304, 12, 1)]
HEADS = [(1000, 256, 1), (5003, 256, 63), (40001, 128, 65), (40000, 128, 130), (40010, 128, 200), (20000, 256, 257),
         (126464, 128, 33), (126464, 128, 64), (5003, 208, 131),
         # 128 ids split over two waves, 128, 192 and 256 tokens: several units per workgroup, partly filled columns
         (152064, 512, 33), (152064, 512, 128), (16010, 512, 193), (32003, 1024, 65),
         (24001, 2048, 129), (24001, 4096, 600), (16010, 4096, 257), (32003, 2048, 189), (32003, 4096, 233), (6001, 512, 769)]


def _plans(dcl):
    layer, head = set(), set()
    for d, F, H, T in LAYERS:
        hd = 64 * H
        for nw, k, split in ((3 * hd, d, 1), (d, hd, 4), (2 * F, d, 1), (d, F, 4)):
            layer.add(dcl.dcl_debug_gemm_plan(nw, T, k, False, split)["cfg"])
    for V, d, n in HEADS:
        head.add(dcl.dcl_debug_gemm_plan(V, n, d, True, 1)["cfg"])
    return layer, head


def test_shapes_cover_every_configuration():
    import paper_2607_20467_amd as dcl
    layer, head = _plans(dcl)
    want = set(range(20)) - {6, 14}
    assert layer >= want, f"configurations {sorted(want - layer)} not covered"
    assert head >= {0, 3, 4, 5, 6, 11, 13, 14, 19}, f"head configurations covered: {sorted(head)}"


def _geom(d, F, H, V=512):
    return dataclasses.replace(synth.TINY, name="tiles", n_layers=1, d_model=d, n_heads=H, n_kv_heads=H, head_dim=64,
                               d_ffn=F, vocab=V, mask_id=V - 1, weight_dtype="bf16")


def _weights(g, gen):
    import torch
    out = []
    for name, shape, kind in synth.tensor_specs(g):
        if kind == "bias":
            out.append(None)
        elif kind == "gain":
            out.append(torch.ones(shape, dtype=torch.bfloat16, device="cuda"))
        else:
            out.append((torch.randn(shape, generator=gen, device="cuda") * 0.05).to(torch.bfloat16))
    return out


def _check(name, got, want, bound, bf16):
    tol = bound + (want.abs() * 2.0 ** -8 if bf16 else 0)
    bad = ~((got.double() - want).abs() <= tol)          # NaN counts as bad
    assert not bool(bad.any()), f"{name}: {int(bad.sum())} of {bad.numel()} elements outside the bound"


@pytest.mark.gpu
@pytest.mark.parametrize("d,F,H,T", LAYERS)
def test_layer_tiles(d, F, H, T):
    import torch
    import paper_2607_20467_amd as dcl
    print(f"case layer d {d} F {F} H {H} T {T}", flush=True)
    g = _geom(d, F, H)
    gen = torch.Generator(device="cuda").manual_seed(d + F + T)
    w = _weights(g, gen)
    run = dcl.Runner(g, w, max_positions=2048, rope_enabled=False)
    hd, Sp = 64 * H, (T + 7) // 8 * 8
    r = torch.randn((T, d), generator=gen, device="cuda")
    i16, f32 = torch.int16, torch.float32
    taps = {k: torch.full((n,), -1, dtype=t, device="cuda") for k, n, t in
            (("u", T * d, i16), ("q", T * hd, i16), ("k", T * hd, i16), ("v", hd * Sp, i16), ("o", T * hd, i16),
             ("r_mid", T * d, f32), ("u2", T * d, i16), ("a", T * F, i16), ("r_out", T * d, f32))}
    ws, n = run.workspace(1, T)
    dcl.dcl_debug_layer(run.model, 1, T, None, 0, r, taps, ws, n)
    b = {k: (v.view(torch.bfloat16) if v.dtype == i16 else v).double() for k, v in taps.items()}
    wq, wk, wv, _, _, _, wo, wg, wu, wd = (None if x is None else x.double() for x in w[1:11])

    def proj(x, m, extra=2):
        return x @ m.t(), (x.shape[1] + extra) * 2.0 ** -23 * (x.abs() @ m.abs().t())
    u, o, u2, a = b["u"].view(T, d), b["o"].view(T, hd), b["u2"].view(T, d), b["a"].view(T, F)
    for name, m in (("q", wq), ("k", wk)):
        _check(name, b[name].view(H, T, 64).transpose(0, 1).reshape(T, hd), *proj(u, m), True)
    v = b["v"].view(hd, Sp)
    _check("v", v[:, :T].t(), *proj(u, wv), True)
    assert bool((v[:, T:] == 0).all()), "v padding"
    y, e = proj(o, wo, 6)
    _check("r_mid", b["r_mid"].view(T, d), r.double() + y, e + (hd + 6) * 2.0 ** -23 * r.double().abs(), False)
    (gt, eg), (up, eu) = proj(u2, wg), proj(u2, wu)
    s = torch.nn.functional.silu(gt)
    _check("a", a, s * up, 1.1 * eg * up.abs() + s.abs() * eu + eg * eu + (s * up).abs() * (gt.abs() + 8) * 2.0 ** -21,
           True)
    y, e = proj(a, wd, 6)
    r_mid = b["r_mid"].view(T, d)
    _check("r_out", b["r_out"].view(T, d), r_mid + y, e + (F + 6) * 2.0 ** -23 * r_mid.abs(), False)


@pytest.mark.gpu
@pytest.mark.parametrize("d,F,H,T", [(1024, 4096, 16, 64), (1024, 4096, 16, 200), (2048, 3072, 16, 768)])
def test_residual_stream_is_rounded_once_per_projection(d, F, H, T):
    """The K slices of a residual GEMM are small beside the stream: added up first, the sum rounds r once. One rounding
    of values with uniform mantissas is a relative 2-norm error of 2.2e-8 to 2.6e-8 (2^-23 sqrt(1 / 28) for one
    binade); two roundings of r would be 3.2e-8 at least, four slices one by one 4.5e-8."""
    import torch
    import paper_2607_20467_amd as dcl
    g = _geom(d, F, H)
    gen = torch.Generator(device="cuda").manual_seed(d + T)
    w = _weights(g, gen)
    w[7], w[10] = w[7] * 2.0 ** -5, w[10] * 2.0 ** -7
    splits = [dcl.dcl_debug_gemm_plan(d, T, k, False, 4)["nsplit"] for k in (64 * H, F)]
    assert max(splits) >= 3, splits
    run = dcl.Runner(g, w, max_positions=1024, rope_enabled=False)
    r = torch.randn((T, d), generator=gen, device="cuda")
    taps = {"o": torch.empty(T * 64 * H, dtype=torch.int16, device="cuda"),
            "a": torch.empty(T * F, dtype=torch.int16, device="cuda"), "r_mid": torch.empty_like(r),
            "r_out": torch.empty_like(r)}
    ws, n = run.workspace(1, T)
    dcl.dcl_debug_layer(run.model, 1, T, None, 0, r, taps, ws, n)
    for x, m, before, after in (("o", w[7], r, "r_mid"), ("a", w[10], taps["r_mid"], "r_out")):
        want = before.double() + taps[x].view(torch.bfloat16).view(T, -1).double() @ m.double().t()
        err = float((taps[after].double() - want).norm() / want.norm())
        assert err <= 2.9e-8, f"{after}: {err:.2e}"


# gates around the ends of silu's range in float32 (its denominator passes 2^126 at -87.3 and the largest float at
# -88.7), beside infinities and ordinary ones; 89 ids a round, so every row of a fragment meets every gate
GATES = [float("inf"), -88.5, 88.5, -88.0, 3e38, -87.5, 0.0, -87.0, 1e-30, -86.5, -1.0, -89.0, 2.0, -200.0, -0.0, -3e38,
         1e38] + [(i - 36) / 4.0 for i in range(72)]


@pytest.mark.gpu
@pytest.mark.parametrize("T", [5, 64, 129, 200, 513])
def test_swiglu_gates_at_the_ends_of_the_range(T):
    """g / (1 + e^-g) of given gates: +inf stays +inf and leaves its neighbours alone, and the quotients past 2^126 keep
    their bits (relative error of the float32 exponential and quotient as in test_layer_tiles)."""
    import torch
    import paper_2607_20467_amd as dcl
    d, F = 384, 6144
    g = _geom(d, F, 1)
    w = _weights(g, torch.Generator(device="cuda").manual_seed(T))
    w[7].zero_()                                            # W_o: the residual stream reaches the MLP unchanged
    gates = torch.tensor([GATES[i % len(GATES)] for i in range(F)], dtype=torch.float64).to(torch.bfloat16).cuda()
    up = torch.tensor([[1.0, -0.5, 3.0][i % 3] for i in range(F)], dtype=torch.float64).to(torch.bfloat16).cuda()
    w[8].zero_()
    w[9].zero_()
    w[8][:, 0], w[9][:, 0] = gates, up
    run = dcl.Runner(g, w, max_positions=2048, rope_enabled=False)
    taps = {k: torch.full((T * n,), -1, dtype=torch.int16, device="cuda") for k, n in (("u2", d), ("a", F))}
    ws, n = run.workspace(1, T)
    dcl.dcl_debug_layer(run.model, 1, T, None, 0, torch.ones((T, d), device="cuda"), taps, ws, n)
    assert bool((taps["u2"].view(torch.bfloat16) == 1).all())
    a = taps["a"].view(torch.bfloat16).view(T, F).double()
    gt = gates.double()
    den = 1 + torch.exp(-gt)
    den[den > torch.finfo(torch.float32).max] = float("inf")   # the float32 denominator
    want = gt / den * up.double()
    inf = gt.isinf()
    assert bool((a[:, inf] == want[inf]).all()), "silu(+inf) up"
    big = want.abs() > torch.finfo(torch.bfloat16).max
    bad = ~((a - want).abs() <= want.abs() * ((gt.abs() + 8) * 2.0 ** -21 + 2.0 ** -8))      # NaN counts as bad
    bad[:, inf | big] = False
    assert not bool(bad.any()), f"gates {gt[bad.any(0)].unique().tolist()} outside the bound"


@pytest.mark.gpu
@pytest.mark.parametrize("V,d,n", HEADS)
def test_head_tiles(V, d, n):
    import torch
    import paper_2607_20467_amd as dcl
    print(f"case head V {V} d {d} n {n}", flush=True)
    g = _geom(d, 16, 1, V)
    gen = torch.Generator(device="cuda").manual_seed(V + d + n)
    w = _weights(g, gen)
    run = dcl.Runner(g, w, max_positions=16)
    hidden = torch.randn((n, d), generator=gen, device="cuda").to(torch.bfloat16)
    st = run.score_hidden(hidden)
    logits = hidden.double() @ w[-1].double().t()
    top = logits.topk(2, -1)
    lse = logits.logsumexp(-1)
    clear = top.values[:, 0] - top.values[:, 1] > TIE_GAP
    assert bool((st["top1"][clear].long() == top.indices[:, 0][clear]).all())
    assert float((st["lse"].double() - lse).abs().max()) <= LOGIT_TOL
    for key, i in (("conf", 0), ("p2", 1)):
        assert float((st[key].double() - torch.exp(top.values[:, i] - lse)).abs().max()) <= CONF_TOL, key
    p = torch.softmax(logits, -1)
    H = lse - (p * logits).sum(-1)
    assert float((st["entropy"].double() - H).abs().max()) <= LOGIT_TOL


@pytest.mark.gpu
@pytest.mark.parametrize("V,B,S,prompt", [(40010, 1, 608, 0), (40010, 1, 608, 48), (40010, 1, 608, 383), (40010, 1, 608, 448),
                                          (40010, 1, 608, 575), (40010, 1, 608, 607), (40010, 1, 608, 608), (40010, 4, 152, 96),
                                          (40010, 7, 640, 0), (40010, 7, 640, 575),
                                          (12001, 2, 190, 0), (12001, 2, 190, 93), (12001, 2, 190, 190)])
def test_step_head_tiles_chosen_by_the_scored_rows(V, B, S, prompt):
    """A step's head where the scored rows, counted on the device, choose the tokens per tile (192 for 560 or 160, 256 for
    608 or 225 of 608) or the number of 128 x 192 tiles. Statistics of the step against float64 on its own hidden states, none scored and
    counts past the last choice included; the rows of other numbers keep their sentinels."""
    import torch
    import paper_2607_20467_amd as dcl
    d, R = 128, B * (S - prompt)
    assert dcl.dcl_debug_gemm_plan(V, B * S, d, 2)["cfg"] == (3 if V == 40010 else 19)
    g = _geom(d, 16, 1, V)
    gen = torch.Generator(device="cuda").manual_seed(R)
    w = _weights(g, gen)
    run = dcl.Runner(g, w, max_positions=1024)
    tok = torch.randint(0, V - 2, (B, S), generator=gen, device="cuda", dtype=torch.int32)
    tok[:, prompt:] = g.mask_id
    st = run.step(tok, torch.full((B,), prompt, dtype=torch.int32, device="cuda"), S)
    scored = torch.zeros((B, S), dtype=torch.bool, device="cuda")
    scored[:, prompt:] = True
    assert bool((st["top1"][~scored] == -1).all()) and bool((st["conf"][~scored] == -1).all())
    if R == 0:
        return
    rows = scored.view(-1).nonzero().view(-1).to(torch.int32)
    hidden = run.logits(tok, rows[:512], with_hidden=True)[1].view(torch.bfloat16).double()
    logits = hidden @ w[-1].double().t()
    top, lse = logits.topk(2, -1), logits.logsumexp(-1)
    got = {k: v[scored][:512] for k, v in st.items()}
    clear = top.values[:, 0] - top.values[:, 1] > TIE_GAP
    assert bool((got["top1"][clear].long() == top.indices[:, 0][clear]).all())
    assert float((got["lse"].double() - lse).abs().max()) <= LOGIT_TOL
    for key, i in (("conf", 0), ("p2", 1)):
        assert float((got[key].double() - torch.exp(top.values[:, i] - lse)).abs().max()) <= CONF_TOL, key
    # every scored row has statistics, the last ones as the rest
    last = run.logits(tok, rows[-1:])[0].double()
    assert float((st["lse"][scored][-1].double() - last.logsumexp(-1)).abs()) <= LOGIT_TOL


@pytest.mark.gpu
@pytest.mark.parametrize("n", [20, 129])
def test_head_ties_and_non_finite_logits(n):
    """Equal logits rank by id wherever the equal ids sit (one lane, two lanes of a token, two vocabulary tiles),
    a -inf logit takes no part, and a row with a NaN logit leaves the other rows alone."""
    import torch
    import paper_2607_20467_amd as dcl
    V, d = 4000, 256
    g = _geom(d, 16, 1, V)
    gen = torch.Generator(device="cuda").manual_seed(n)
    w = _weights(g, gen)
    best = torch.full((d,), 0.25, dtype=torch.bfloat16, device="cuda")
    groups = ([65, 66], [200, 204], [385, 401], [600, 2600], [1000, 1016, 3999])
    hidden = (torch.rand((n, d), generator=gen, device="cuda") + 0.5).to(torch.bfloat16)
    for ids in groups:
        m = [x.clone() if x is not None else None for x in w]
        m[-1][ids] = best
        m[-1][17, 3] = -torch.inf                       # hidden[:, 3] > 0: logit -inf in every row
        h = hidden.clone()
        h[n - 1, 5] = torch.nan
        st = dcl.Runner(g, m, max_positions=16).score_hidden(h)
        assert st["top1"][:n - 1].tolist() == [ids[0]] * (n - 1)
        assert st["top2"][:n - 1].tolist() == [ids[1]] * (n - 1)
        logits = h[:n - 1].double() @ m[-1].double().t()
        conf = torch.softmax(logits, -1)[:, ids[0]]
        assert float((st["conf"][:n - 1].double() - conf).abs().max()) <= CONF_TOL
        assert bool((st["conf"][:n - 1] == st["p2"][:n - 1]).all())
        assert bool(st["conf"][n - 1].isnan())
