"""Edges of the fp32 products' small tiles (32 x 32, 32 deep): rows, columns and depths just below, at and above a tile,
depths that allow 16-byte loads and depths that do not, head sizes with and without them, and a batch large enough for
the 64 x 64 tiles.  Bound of the fp32 path: 1e-4 of the largest logit."""
import pytest

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth
from tests import parity as Pz

pytestmark = pytest.mark.gpu

CASES = [
    # (heads, head size, FFN, vocabulary, batch, rows)
    (1, 32, 31, 33, 1, 1), (1, 32, 32, 64, 1, 32), (1, 34, 33, 65, 1, 33), (3, 10, 47, 100, 2, 31), (3, 22, 64, 95, 1, 65),
    (2, 36, 130, 129, 3, 17), (4, 64, 512, 1000, 4, 150),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_f32_edges(case):
    H, Dh, F, V, B, T = CASES[case]
    m = synth.ModelShape(2, H * Dh, H, Dh, F, V, V - 1, V - 2, dtype="fp32")
    weights = synth.make_weights(m, 440 + case, "cpu")
    ora = Pz.oracle_model(m, weights)
    eng = Bd.Engine(m, Pz.to_dev(weights), B, max(T, 2))
    X = synth.make_prompt(460 + case, B, T, V - 2, "cpu")
    got = eng.forward(X.cuda()).cpu().numpy()
    for b in range(B):
        assert Pz.rel_err(got[b], ora.forward(X[b].numpy())) < 1e-4, b
