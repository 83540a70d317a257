"""Edges of the bf16 attention kernel through one-layer models: query groups of 32 and key tiles of 64 that are filled,
missed by one and exceeded by one; every split of a workgroup (one and two key ranges, 32 to 256 queries) at both head
sizes; scores that grow along the keys, so that the reference of the exponents has to follow the running maximum after
the first tile.  Bound of the other bf16 forwards: 2e-2 of the largest logit."""
import numpy as np
import pytest
import torch

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth
from tests import parity as Pz

pytestmark = pytest.mark.gpu

CASES = [
    # (heads, head size, batch, rows): 1 / 2 wavefronts and ranges for few rows, 2 x 2, 4 x 2, 8 x 1
    (2, 64, 1, 1), (2, 128, 1, 31), (2, 64, 1, 33), (1, 128, 2, 64), (2, 64, 1, 65), (2, 128, 1, 127), (1, 64, 3, 129),
    (8, 128, 9, 257), (16, 64, 8, 250), (32, 64, 1, 1100), (16, 128, 1, 2100),
]


@pytest.mark.parametrize("sharp", [1.0, 6.0])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_attention_edges(case, sharp):
    H, Dh, B, T = CASES[case]
    m = synth.ModelShape(1, H * Dh, H, Dh, 64, 300, 299, 298, dtype="bf16")
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
