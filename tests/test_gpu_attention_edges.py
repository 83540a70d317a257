"""Edges of the bf16 attention kernel through two-layer models (all rows in the first layer, the wanted ones in the
second): query groups of 32 and key tiles of 64 that are filled, missed by one and exceeded by one; every dealing of the
key ranges to a workgroup's wavefronts at both head sizes; scores of tens, so that the running maximum moves from tile
to tile.  Block rows over a store: key counts around multiples of a tile, ranges of unequal length and empty ones, keys
dealt to several workgroups.  Bound of the other bf16 forwards: 2e-2 of the largest logit."""
import numpy as np
import pytest
import torch

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth
from tests import parity as Pz

pytestmark = pytest.mark.gpu

CASES = [
    # (heads, head size, batch, rows); query groups x ranges side by side x ranges in turn:
    (2, 64, 1, 1), (2, 128, 1, 31),                                              # 1 x 2 x 2
    (2, 64, 1, 33), (1, 128, 2, 64), (2, 64, 1, 65), (2, 128, 1, 127), (1, 64, 3, 129), (16, 64, 8, 250),   # 2 x 2 x 2
    (8, 64, 70, 40), (8, 128, 33, 64),                                           # 2 x 1 x 4
    (8, 128, 9, 257), (16, 64, 9, 250),                                          # 4 x 1 x 4
    (32, 64, 1, 1100), (16, 128, 1, 2000),                                       # 4 x 2 x 1
    (32, 64, 2, 1100), (16, 128, 1, 2100),                                       # 4 x 1 x 2
]


@pytest.mark.parametrize("sharp", [1.0, 6.0])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_attention_edges(case, sharp):
    H, Dh, B, T = CASES[case]
    m = synth.ModelShape(2, H * Dh, H, Dh, 64, 300, 299, 298, dtype="bf16")
    weights = synth.make_weights(m, 340 + case, "cpu")
    for name in ("layers.0.wq", "layers.0.wk"):      # sharp: scores of tens, maxima that move from tile to tile
        weights[name] = (weights[name].float() * sharp).to(weights[name].dtype)
    ora = Pz.oracle_model(m, weights, gemm_input="bf16")
    eng = Bd.Engine(m, Pz.to_dev(weights), B, max(T, 2))
    X = synth.make_prompt(360 + case, B, T, 298, "cpu")
    rows = min(T, 70)
    got = eng.forward(X.cuda(), T - rows, rows).cpu().numpy()
    for b in {0, B - 1}:
        ref = ora.forward(X[b].numpy())[T - rows:]
        assert Pz.rel_err(got[b], ref) < 2e-2, b


@pytest.mark.parametrize("H,Dh,B,block,T", [
    (2, 64, 1, 31, 65), (2, 128, 2, 31, 129), (2, 64, 2, 33, 129), (2, 128, 1, 64, 193), (1, 64, 3, 64, 320), (2, 128, 1, 32, 383),
    (8, 64, 70, 33, 193), (8, 128, 33, 64, 321),               # more than a round of workgroups: the ranges in turn
    (2, 64, 1, 32, 520), (2, 128, 2, 64, 577), (2, 64, 1, 33, 1100), (8, 128, 3, 31, 700),   # keys dealt to several workgroups
    (2, 64, 2, 100, 500), (2, 128, 1, 128, 577),               # blocks of more than 64 rows
])
def test_block_rows_over_a_store(H, Dh, B, block, T):
    # the first step after a dual-cache rebuild sees nothing stale: its logits are the full forward's
    m = synth.ModelShape(2, H * Dh, H, Dh, 64, 300, 299, 298, dtype="bf16")
    weights = synth.make_weights(m, 41, "cpu")
    ora = Pz.oracle_model(m, weights, gemm_input="bf16")
    eng = Bd.Engine(m, Pz.to_dev(weights), B, T, prefix_cache=True)
    X = synth.make_prompt(42, B, T, 298, "cpu")
    cfg = Bd.Engine.cfg_struct(block, block, 0.5, dual_cache=True)
    state = torch.zeros((B, 3), dtype=torch.int32, device="cuda")
    got = eng.denoise_step(X.cuda(), T - block, state, synth.make_filter(3, block, 32, "cuda"), cfg, want_logits=True)["logits"]
    for b in sorted({0, B - 1}):
        assert Pz.rel_err(got[b].cpu().numpy(), ora.forward(X[b].numpy())[T - block:]) < 2e-2, b


@pytest.mark.parametrize("H,Dh,block", [(32, 64, 64), (32, 64, 40), (16, 128, 64), (16, 128, 32), (16, 128, 17)])
def test_block_rows_are_the_same_bits_in_every_batch(H, Dh, block):
    # block-only steps over a dual cache, more than 256 rows in every batch (up to there the projections' K ranges follow
    # the row count) and at least 128 workgroups (below, the keys are dealt to several): a sequence's logits may not
    # depend on how many others are in the launch, whatever that does to the choice of kernel
    B, n, P = max(48, -(-600 // H) + 8), 3, 3 * block + 5
    m = synth.ModelShape(1, H * Dh, H, Dh, 128, 300, 299, 298, dtype="bf16")
    eng = Bd.Engine(m, synth.make_weights(m, 31, "cuda"), B, P + n * block, prefix_cache=True)
    flt = synth.make_filter(3, block, 32, "cuda")
    X = synth.make_prompt(32, B, P + n * block, 298, "cuda")
    cfg = Bd.Engine.cfg_struct(n * block, block, 0.5, dual_cache=True)
    def logits(first, count):
        state = torch.tensor([[1, 0, 0]] * count, dtype=torch.int32, device="cuda")
        return eng.denoise_step(X[first:first + count].clone(), P, state, flt, cfg, want_logits=True)["logits"]
    every = logits(0, B)
    few = max(-(-257 // block), -(-128 // H))
    for first, count in ((0, few), (B - few, few), (1, 512 // H - 1), (2, 512 // H), (3, B - 5)):
        if count >= few:
            assert torch.equal(logits(first, count), every[first:first + count]), (first, count)
