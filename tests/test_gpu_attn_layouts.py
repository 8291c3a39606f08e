"""Every attention layout at the edges of its tiles: query counts one past or short of a workgroup's, key counts one
past or short of a tile, key groups without keys, cached prefixes that end inside a chunk or a tile, against float64.

dcl_debug_layer's own q, k, v (taps) give the reference. A probability is exp2(x) of a float32 score x whose terms
and rounding err by at most (dh + 4) 2^-23 sum |q k| scale (log2 units, times ln 2 for the probability's relative
error), and the sums of P v and of P over n keys err by at most (n + 32) 2^-23 of sum P |v|; a bfloat16 store adds
half an ulp, at most 2^-8 of the value.
"""
import dataclasses
import math

import pytest

import synth

# (head_dim, heads, kv heads, batch, tokens, cached): layouts by (query waves, keys), see launch_attention
CASES = [
    (128, 4, 2, 1, 17, 0), (128, 4, 4, 1, 65, 0), (128, 4, 2, 2, 33, 331), (128, 2, 1, 1, 1, 96),       # few
    (64, 4, 4, 1, 96, 0), (64, 4, 2, 3, 33, 45), (64, 8, 8, 1, 64, 0), (64, 16, 4, 9, 31, 70),
    (128, 16, 4, 5, 49, 8), (128, 16, 16, 5, 33, 9), (128, 16, 4, 1, 799, 0), (128, 16, 4, 2, 449, 0),  # 2 x 1 x 2
    (128, 16, 8, 2, 512, 0), (128, 16, 4, 9, 65, 290), (128, 16, 16, 20, 30, 331), (128, 16, 8, 32, 19, 338),
    (128, 16, 4, 16, 17, 333), (128, 16, 4, 8, 50, 333), (128, 32, 4, 2, 97, 1217), (128, 16, 4, 3, 161, 0),
    (128, 16, 16, 15, 33, 270), (128, 16, 16, 9, 41, 331), (128, 16, 4, 5, 180, 322), (128, 16, 16, 9, 50, 111),  # 4 x 1 x 2
    (128, 32, 4, 6, 289, 35), (128, 16, 8, 20, 131, 260), (128, 16, 4, 64, 17, 331),
    (128, 16, 8, 9, 40, 71), (128, 16, 4, 15, 47, 0), (128, 16, 4, 3, 700, 0), (128, 16, 8, 33, 19, 338),  # 4 x 1 x 1
    (128, 16, 4, 3, 977, 0), (128, 16, 16, 4, 577, 0), (128, 16, 4, 9, 50, 110), (128, 16, 16, 60, 3, 23),
    (128, 16, 4, 65, 17, 331), (128, 16, 4, 23, 129, 331), (128, 16, 4, 3, 160, 0),
    (128, 16, 4, 2, 577, 0), (128, 16, 8, 3, 331, 13), (128, 16, 4, 4, 512, 0),                         # 2 x 2 x 2
    (128, 16, 4, 4, 833, 0), (128, 16, 4, 13, 200, 90), (128, 32, 4, 13, 66, 332), (128, 16, 4, 13, 193, 0),  # 4 x 2 x 1
    (64, 16, 4, 1, 641, 0), (64, 16, 8, 2, 805, 0), (64, 16, 4, 4, 130, 333), (64, 16, 2, 5, 577, 9),    # 64-key tiles
    (64, 4, 2, 70, 1, 15),                                        # more carried rows in a GEMM tile than threads
]


@pytest.mark.gpu
@pytest.mark.parametrize("dh,H,Hkv,B,S,P", CASES)
def test_attention_layout(dh, H, Hkv, B, S, P):
    import torch
    import paper_2607_20467_amd as dcl
    print(f"case dh {dh} H {H}/{Hkv} B {B} S {S} P {P}", flush=True)
    d = 256
    g = dataclasses.replace(synth.TINY, name="attn", n_layers=1, d_model=d, n_heads=H, n_kv_heads=Hkv, head_dim=dh,
                            d_ffn=64, vocab=512, mask_id=511, weight_dtype="bf16")
    gen = torch.Generator(device="cuda").manual_seed(dh + H + B + S + P)
    w = []
    for name, shape, kind in synth.tensor_specs(g):
        w.append(None if kind == "bias" else torch.ones(shape, dtype=torch.bfloat16, device="cuda") if kind == "gain"
                 else (torch.randn(shape, generator=gen, device="cuda") * 0.08).to(torch.bfloat16))
    run = dcl.Runner(g, w, max_positions=4096)
    koff, Pc = P % 8, (P + 15) // 8 * 8
    Sk = S + koff
    Sp = (Sk + 7) // 8 * 8
    kv = None
    if P:
        def cache(*shape):
            return torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
        kc, vc = cache(B, Hkv, Pc, dh), cache(B, Hkv, dh, Pc)
        kc[:, :, P:], vc[..., P:] = float("nan"), float("nan")   # past the prefix: never used
        kv = ([kc], [vc], P, Pc)
    r = torch.randn((B * S, d), generator=gen, device="cuda")
    taps = {k: torch.full((n,), -1, dtype=torch.int16, device="cuda") for k, n in
            (("q", B * S * H * dh), ("k", B * Sk * Hkv * dh), ("v", B * Hkv * dh * Sp), ("o", B * S * H * dh))}
    ws, n = run.workspace(B, S, P)
    dcl.dcl_debug_layer(run.model, B, S, kv, 0, r, taps, ws, n)
    b = {k: v.view(torch.bfloat16) for k, v in taps.items()}
    k, v = b["k"].view(B, Hkv, Sk, dh), b["v"].view(B, Hkv, dh, Sp)
    if P:   # the newest P mod 8 cached keys and values stand in front of the fresh ones
        assert torch.equal(k[:, :, :koff], kc[:, :, P - koff:P]) and torch.equal(v[..., :koff], vc[..., P - koff:P])
        k = torch.cat((kc[:, :, :P - koff], k), 2)
        v = torch.cat((vc[..., :P - koff], v[..., :Sk]), 3)
    q, k, v = b["q"].view(B, H, S, dh).double(), k.double(), v[..., :P + S].double().transpose(2, 3)
    got = b["o"].view(B, S, H, dh).double()
    for h in range(H):
        kh, vh = k[:, h // (H // Hkv)].contiguous(), v[:, h // (H // Hkv)].contiguous()
        kt = kh.transpose(1, 2).contiguous()
        p = torch.softmax(torch.bmm(q[:, h], kt) / math.sqrt(dh), -1)
        rel = torch.bmm(q[:, h].abs(), kt.abs()) * ((dh + 4) * 2.0 ** -23 / math.sqrt(dh)) + (P + S + 32) * 2.0 ** -23
        want, err = torch.bmm(p, vh), 2 * torch.bmm(p * rel, vh.abs())
        # the normalising sum's own relative error, the average of the keys' ones
        err += want.abs() * (p * rel).sum(-1, keepdim=True)
        bad = ~((got[:, :, h] - want).abs() <= err + want.abs() * 2.0 ** -8)     # NaN counts as bad
        assert not bool(bad.any()), f"head {h}: {int(bad.sum())} elements outside the bound"
