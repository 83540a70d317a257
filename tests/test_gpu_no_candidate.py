"""Rows whose logits are all -inf or no numbers: the greedy token is still a token, and not the mask id.  (What is committed
indexes the embedding in the next step.)"""
import pytest
import torch

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,V,mask", [("fp32", 64, 100, 99), ("fp32", 64, 70, 0), ("bf16", 64, 300, 299), ("bf16", 128, 130, 0)])
@pytest.mark.parametrize("value", [float("-inf"), float("nan")])
@pytest.mark.parametrize("B,s", [(1, 32), (3, 64)])
def test_a_token_is_committed_all_the_same(dtype, d, V, mask, value, B, s):
    m = synth.ModelShape(1, d, d // 64, 64, 64, V, mask, V - 2, dtype=dtype)
    w = synth.make_weights(m, 830, "cuda")
    # the first feature of the last hidden row is positive, and the head takes it alone: value times it
    w["tok_emb"][:, 0] = 100.
    w["final_norm_g"].zero_()
    w["final_norm_g"][0] = 1e3 if dtype == "fp32" else 256.
    w["lm_head"].zero_()
    w["lm_head"][:, 0] = value if value != value else -3e38
    P, G = 8, 2 * s
    eng = Bd.Engine(m, w, B, P + G)
    X = synth.make_prompt(831, B, P + G, V - 2, "cuda").clamp_(min=1)
    X[:, P:] = m.mask_id
    state = torch.zeros((B, 3), dtype=torch.int32, device="cuda")
    out = eng.denoise_step(X, P, state, synth.make_filter(832, s, 32, "cuda"), Bd.Engine.cfg_struct(G, s, 0.5), want_logits=True)
    logits = out["logits"]
    assert (torch.isnan(logits) if value != value else logits == value).all()
    lowest = 1 if mask == 0 else 0
    assert (out["pred"] == lowest).all()
    assert ((X >= 0) & (X < V)).all()
    assert ((X[:, P:P + s] != m.mask_id).sum(1) >= 1).all()
