"""The fp32 products and attention at their edges: head sizes below, at and between the padded ones, depths that leave K ranges
ragged or empty, keys that leave a wavefront without any, and batches on either side of the large tiles, where a
sequence's logits must not change.  Bound against the oracle: 1e-4 of the largest logit (the fp32 path's)."""
import pytest
import torch

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth
from tests import parity as Pz

pytestmark = pytest.mark.gpu

CASES = [
    # (heads, head size, FFN, vocabulary, batch, rows)
    (1, 2, 5, 33, 1, 2), (2, 6, 17, 40, 1, 16), (1, 16, 15, 31, 2, 17), (2, 66, 48, 64, 1, 49), (1, 130, 100, 97, 1, 130),
    (1, 256, 64, 130, 2, 70), (2, 128, 260, 200, 1, 33),
]


def model(H, Dh, F, V):
    return synth.ModelShape(2, H * Dh, H, Dh, F, V, V - 1, V - 2, dtype="fp32")


@pytest.mark.parametrize("case", CASES)
def test_edges_match_oracle(case):
    H, Dh, F, V, B, T = case
    m = model(H, Dh, F, V)
    weights = synth.make_weights(m, 510, "cpu")
    ora = Pz.oracle_model(m, weights)
    eng = Bd.Engine(m, Pz.to_dev(weights), B, max(T, 2))
    X = synth.make_prompt(511, B, T, V - 2, "cpu")
    got = eng.forward(X.cuda()).cpu().numpy()
    for b in range(B):
        assert Pz.rel_err(got[b], ora.forward(X[b].numpy())) < 1e-4, b


def test_large_tiles_give_the_bits_of_small_ones():
    # 8 x 512 rows: Q/K/V, gate/up and the head (8 x 256 rows) in 64 x 64 tiles; one sequence alone: 16 x 32 ones
    m = model(6, 64, 512, 4100)
    weights = synth.make_weights(m, 520, "cuda")
    X = synth.make_prompt(521, 8, 512, m.vocab - 2, "cuda")
    eng = Bd.Engine(m, weights, 8, 512)
    whole = eng.forward(X, 100, 256)
    for b in (0, 5):
        assert torch.equal(eng.forward(X[b:b + 1].contiguous(), 100, 256)[0], whole[b]), b
    ora = Pz.oracle_model(m, {k: v.cpu() for k, v in weights.items()})
    assert Pz.rel_err(whole[3].cpu().numpy(), ora.forward(X[3].cpu().numpy())[100:356]) < 1e-4
