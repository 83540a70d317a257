"""Precision of the attention probabilities in the bf16 path, seen through the logits of a one-layer model.

Every query of a head gives one heavy key (the last position) a third to two thirds of its weight and shares the rest
among a hundred light keys of nearly equal scores, which lie between keys that count for nothing; one value feature is
+1 at the heavy key and -c at the light ones, c such that the exact output is next to zero.  What is left there is the
rounding of the probabilities to bf16: the heavy key is the running maximum when its tile is reached, so its probability
has to be exactly 1, and the light keys' roundings average out.  With n light keys of weight w / n each, rounded by at
most 2^-9 and independently of one another, the output's standard deviation is w * 2^-9 / sqrt(3 n), w <= 2/3;
the bound is five of these (and 2e-5 for the roundings behind the attention, which are relative to an output of 2e-3).
A heavy key whose own probability is rounded misses it several times over.

The model: embeddings of +-1 (token t is -1 at feature t alone, so every weight row gives each token any value), one query /
key feature per head whose rotation angle vanishes, output projection 1024 times the identity on the value features, no
FFN, LM head the identity.  A second value feature is 1 everywhere and fixes the final norm."""
import math

import pytest
import torch

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth

pytestmark = pytest.mark.gpu

GAIN, LIGHT = 1024.0, 100


def bound():
    return 5 * 2 / 3 * 2.0 ** -9 / math.sqrt(3 * LIGHT) + 2e-5


def crafted_model(H, Dh, T):
    d = H * Dh
    assert T <= d - 3
    m = synth.ModelShape(1, d, H, Dh, 64, d + 2, d, d + 1, rope_base=1e30, rms_eps=0.0, dtype="bf16")
    one = d - 1                                    # +1 in the embedding of every token used, as are d - 2 and d - 3
    f = Dh * 5 // 16                               # rotation angle: position * 1e-18
    light = torch.full((T - 1,), -32.0, dtype=torch.float64)
    light[::(T - 1) // LIGHT][:LIGHT] = torch.tensor([(1 + i // 2) / 128 * (1 if i % 2 else -1) for i in range(LIGHT)],
                                                      dtype=torch.float64)
    dark = T - 1 - LIGHT
    w = {k: torch.zeros(s, dtype=torch.float64) for k, s in (("wq", (d, d)), ("wk", (d, d)), ("wv", (d, d)), ("wo", (d, d)))}
    emb = torch.ones(d + 2, d, dtype=torch.float64)
    emb[torch.arange(T), torch.arange(T)] = -1.0
    out = torch.zeros(d, dtype=torch.float64)      # the attention output of every query, exactly
    for h in range(H):
        at = h * Dh
        heavy = round(32 * (math.log(LIGHT) - 0.7 + 1.2 * h / H)) / 32 * (8.0 / math.sqrt(Dh)) ** -1
        heavy = torch.tensor(heavy).bfloat16().item()
        key = torch.cat([light, torch.tensor([heavy], dtype=torch.float64)])
        w["wq"][at + f, one] = 8.0
        w["wk"][at + f, :T] = -key / 2
        w["wk"][at + f, one] = heavy / 2           # the rows' sums, so that token t gets key[t]
        w["wk"][at + f, one - 1], w["wk"][at + f, one - 2] = -16.0 * (dark // 256 * 256), -16.0 * (dark % 256)
        p = torch.softmax(key * 8.0 / math.sqrt(Dh), 0)
        c = (p[-1] / p[:-1].sum()).item()
        a, b = (torch.tensor(v).bfloat16().double() for v in ((1 - c) / 2, -(1 + c) / 2))
        w["wv"][at, one], w["wv"][at, T - 1] = a, b
        w["wv"][at + 1, one] = 1.0
        value = torch.full((T,), (a + b).item(), dtype=torch.float64)
        value[-1] = a - b
        out[at], out[at + 1] = p @ value.bfloat16().double(), 1.0
        w["wo"][at, at] = w["wo"][at + 1, at + 1] = GAIN
    head = torch.zeros(d + 2, d)
    head[:d] = torch.eye(d)
    g, ffn = torch.ones(d).bfloat16(), torch.zeros(64, d).bfloat16()
    weights = {"tok_emb": emb.bfloat16(), "lm_head": head.bfloat16(), "final_norm_g": g, "layers.0.attn_norm_g": g,
               "layers.0.ffn_norm_g": g, "layers.0.w_gate": ffn, "layers.0.w_up": ffn,
               "layers.0.w_down": ffn.t().contiguous(), **{f"layers.0.{k}": v.bfloat16() for k, v in w.items()}}
    for k, v in w.items():
        assert torch.equal(v, weights[f"layers.0.{k}"].double()), k      # every weight is a bf16 number
    return m, weights, emb, out


CASES = [
    # (heads, head size, sequences, positions, block): block 0 a forward, else a step of the last block over a dual cache
    (8, 64, 1, 256, 0), (8, 64, 20, 256, 0), (8, 128, 1, 256, 0), (8, 128, 32, 256, 0), (8, 128, 3, 333, 0),
    (36, 64, 1, 1100, 0), (18, 128, 1, 1900, 0),
    (8, 64, 2, 256, 32), (8, 128, 40, 256, 32), (8, 64, 3, 256, 64), (8, 128, 40, 320, 64), (8, 64, 64, 256, 64),
    (8, 128, 64, 576, 64),
]


@pytest.mark.parametrize("H,Dh,B,T,block", CASES)
def test_the_heaviest_key_is_not_rounded(H, Dh, B, T, block):
    m, weights, emb, out = crafted_model(H, Dh, T)
    eng = Bd.Engine(m, {k: v.cuda() for k, v in weights.items()}, B, T, prefix_cache=block > 0)
    X = torch.arange(T, dtype=torch.int32, device="cuda").repeat(B, 1)
    rows = block or 16
    if block:
        cfg = Bd.Engine.cfg_struct(2 * block, block, 0.5, dual_cache=True)
        state = torch.tensor([[1, 0, 0]] * B, dtype=torch.int32, device="cuda")
        got = eng.denoise_step(X, T - 2 * block, state, synth.make_filter(1, block, 32, "cuda"), cfg, want_logits=True)["logits"]
    else:
        got = eng.forward(X, T - rows, rows)
    e = emb[T - rows:T].cuda()
    hidden = e + GAIN * out.cuda()
    rms = hidden.square().mean(1, keepdim=True).sqrt()
    seen = (got[..., :m.d_model].double() * rms - e) / GAIN
    err = (seen - out.cuda())[..., 0::Dh].abs()
    print(f"largest error {err.max().item():.2e}, bound {bound():.2e}")
    assert err.max().item() < bound()
