"""Numbers beyond the range of fp32 inside the fp32 kernels: what they exclude stays excluded, and the rest is as without them."""
import dataclasses

import pytest
import torch

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth
from tests import parity as Pz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,lo,hi", [(128, 0, 32), (128, 32, 64), (200, 0, 150), (49, 0, 16), (300, 20, 290)])
def test_keys_with_scores_of_minus_infinity_stay_out(T, lo, hi):
    # One head of four features of which the second carries the scores (its rotation is slower than 1e-5 a position).  Keys
    # lo .. hi - 1 are tokens whose product with every query overflows to -inf: whole tiles of them, a wavefront's first
    # ones and all that it has.  The other tokens' scores are zero.
    m = dataclasses.replace(synth.ModelShape(2, 4, 1, 4, 8, 32, 31, 30, dtype="fp32"), rope_base=1e12)
    w = synth.make_weights(m, 810, "cpu")
    emb = w["tok_emb"]
    emb[:] = torch.tensor([1., 0., .5, 0.])
    emb[:, 3] = torch.linspace(-.2, .2, m.vocab)
    emb[16:, 1] = 1.
    w["layers.0.wq"].zero_()
    w["layers.0.wq"][1, 0] = 1e20
    w["layers.0.wk"].zero_()
    w["layers.0.wk"][1, 1] = -1e20
    X = synth.make_prompt(811, 1, T, 16, "cpu")
    X[0, lo:hi] += 14                         # 16 .. 29 from 2 on, the rest 14 and 15
    X[0, lo:hi].clamp_(min=16)
    want = Pz.oracle_model(m, w).forward(X[0].numpy())
    got = Bd.Engine(m, Pz.to_dev(w), 1, T).forward(X.cuda())[0].cpu().numpy()
    assert Pz.rel_err(got, want) < 1e-4
