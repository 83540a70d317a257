"""The products whose wavefronts go in step (64 x 64, 128 x 64 and 128 x 128 tiles): K of one stage up to more than their rings
hold, even and odd numbers of them, row counts around the tiles, sequences that end inside a tile, windows that are no
multiple of four (the transposed value store), and the row-by-row bits against a batch that takes other tiles.  Bound
against the oracle as for the other bf16 forwards: 2e-2 of the largest logit."""
import pytest
import torch

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth
from tests import parity as Pz

pytestmark = pytest.mark.gpu

CASES = [
    # (d, H, Dh, F, B, T)
    (64, 1, 64, 64, 1, 66), (128, 1, 128, 192, 1, 127), (320, 5, 64, 256, 1, 128), (384, 3, 128, 320, 1, 191),
    (448, 7, 64, 448, 1, 193), (512, 4, 128, 1472, 3, 83), (1024, 16, 64, 2816, 1, 221), (1024, 8, 128, 2816, 1, 97),
    (1024, 16, 64, 2816, 2, 206),     # 412 rows: Q/K/V 128 x 64, gate/up 128 x 128, down 64 x 64 in two ranges
    (1344, 21, 64, 1344, 1, 450),     # Q/K/V 128 x 128
    (2048, 16, 128, 4096, 1, 190),
    (1024, 8, 128, 8192, 1, 300),     # K = 8192 above 256 rows: down in four ranges
    (512, 8, 64, 8320, 2, 150),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_edges_match_oracle(case):
    d, H, Dh, F, B, T = CASES[case]
    m = synth.ModelShape(2, d, H, Dh, F, 300, 299, 298, dtype="bf16")
    weights = synth.make_weights(m, 640 + case, "cpu")
    ora = Pz.oracle_model(m, weights, gemm_input="bf16")
    eng = Bd.Engine(m, Pz.to_dev(weights), B, T)
    X = synth.make_prompt(660 + case, B, T, 298, "cpu")
    got = eng.forward(X.cuda())
    assert torch.equal(got, eng.forward(X.cuda()))
    for b in sorted({0, B - 1}):
        assert Pz.rel_err(got[b].cpu().numpy(), ora.forward(X[b].numpy())) < 2e-2, b


@pytest.mark.parametrize("F", [4096, 8192])     # the down projection in two ranges of K and in four
def test_rows_are_the_same_bits_in_large_tiles(F):
    # 270 rows alone (64 x 64 and 128 x 64 tiles) and as one of twelve sequences (256-row tiles with wavefronts in turns)
    m = synth.ModelShape(2, 1024, 8, 128, F, 300, 299, 298, dtype="bf16")
    eng = Bd.Engine(m, synth.make_weights(m, 3, "cuda"), 12, 270)
    X = synth.make_prompt(5, 12, 270, 298, "cuda")
    many = eng.forward(X, 0, 200)
    for b in (0, 7, 11):
        assert torch.equal(eng.forward(X[b:b + 1].contiguous(), 0, 200)[0], many[b]), b
