"""Up to 64 rows: every way that Q/K/V, gate/up and the LM head of few rows can take, at the row counts where their tiles change,
against the oracle.  The widths lie at either side of the lines between the ways."""
import numpy as np
import pytest
import torch

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth
from tests import parity as Pz

pytestmark = pytest.mark.gpu

# (d, H, Dh, F, V): 32 columns to a workgroup, 64 or 96, wider ones, K ranges with a finishing kernel
SHAPES = [(256, 4, 64, 4096, 300), (256, 2, 128, 4160, 129), (128, 2, 64, 8192, 127), (128, 1, 128, 8256, 128), (128, 1, 128, 12288, 300), (128, 1, 128, 12352, 257),
          (1600, 25, 64, 64, 130), (1600, 25, 64, 1984, 130), (2688, 21, 128, 128, 200), (2816, 22, 128, 2048, 200),
          (128, 1, 128, 8320, 130)]       # the last tile of 96 gate/up columns has 32


@pytest.mark.parametrize("case", range(len(SHAPES)))
def test_few_rows_match_the_oracle(case):
    d, H, Dh, F, V = SHAPES[case]
    m = synth.ModelShape(1, d, H, Dh, F, V, V - 1, V - 2, dtype="bf16")
    weights = synth.make_weights(m, 860 + case, "cpu")
    ora = Pz.oracle_model(m, weights, gemm_input="bf16")
    eng = Bd.Engine(m, Pz.to_dev(weights), 2, 64)
    for B, T in ((1, 1), (1, 32), (2, 16), (1, 33), (2, 31), (1, 64)):
        X = synth.make_prompt(870 + T, B, T, V - 2, "cpu")
        got = eng.forward(X.cuda()).cpu().numpy()
        np.testing.assert_array_equal(got, eng.forward(X.cuda()).cpu().numpy())
        assert max(Pz.rel_err(got[b], ora.forward(X[b].numpy())) for b in range(B)) < 2e-2, (B, T)
