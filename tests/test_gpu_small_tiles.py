"""Tiles of narrow models: 64x32, 64x64 one or two to a CU (the last shape: projections of more than 256 tiles), at the widths and
rows on both sides of the lines between them.  Against the oracle, and above 256 rows bit for bit against the same sequence in a
batch, which takes other tiles (below 449 keys: from there on the attention of few workgroups deals the keys among them)."""
import pytest
import torch

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth
from tests import parity as Pz

pytestmark = pytest.mark.gpu

# (d, head size, FFN)
SHAPES = [(256, 64, 704), (512, 128, 1408), (1024, 64, 2816), (1536, 128, 1024), (2816, 128, 704)]


def model(case):
    d, Dh, F = SHAPES[case]
    m = synth.ModelShape(1, d, d // Dh, Dh, F, 200, 199, 198, dtype="bf16")
    return m, synth.make_weights(m, 880 + case, "cpu")


@pytest.mark.parametrize("case", range(len(SHAPES)))
@pytest.mark.parametrize("T", [65, 129, 193, 256, 257, 321])
def test_rows_match_the_oracle(case, T):
    m, weights = model(case)
    eng = Bd.Engine(m, Pz.to_dev(weights), 1, T)
    X = synth.make_prompt(890 + T, 1, T, m.vocab - 2, "cpu")
    got = eng.forward(X.cuda()).cpu().numpy()
    assert Pz.rel_err(got[0], Pz.oracle_model(m, weights, gemm_input="bf16").forward(X[0].numpy())) < 2e-2


@pytest.mark.parametrize("case", range(len(SHAPES)))
@pytest.mark.parametrize("T", [257, 300, 440])
def test_a_sequence_has_the_bits_that_it_has_in_a_batch(case, T):
    m, weights = model(case)
    B = 5
    eng = Bd.Engine(m, Pz.to_dev(weights), B, T)
    X = synth.make_prompt(900 + T, B, T, m.vocab - 2, "cpu").cuda()
    many = eng.forward(X)
    for b in (0, B - 1):
        assert torch.equal(eng.forward(X[b:b + 1])[0], many[b])
