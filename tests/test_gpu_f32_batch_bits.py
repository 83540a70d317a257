"""An fp32 denoising step gives a sequence the same bits whatever batch it is in: logits, confidences, tokens and filter
outputs, with the head's products in large tiles (a batch) and in small ones (a sequence alone), and vocabularies that end in
the first and the second half of a large tile, and on either side of the size from which parts are 64 columns wide."""
import pytest
import torch

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,B,s", [(4100, 8, 128), (4139, 8, 128), (1024, 17, 256), (16320, 6, 48), (16321, 6, 48), (40001, 5, 24)])
def test_step_of_a_batch_gives_the_bits_of_each_sequence_alone(V, B, s):
    m = synth.ModelShape(2, 128, 4, 32, 256, V, V - 1, V - 2, dtype="fp32")
    weights = synth.make_weights(m, 820, "cuda", lm_head_scale=25.0)
    flt = synth.make_filter(821, s, 64, "cuda")
    P, G = 40, 2 * s
    X = synth.make_prompt(822, B, P + G, V - 2, "cuda")
    X[:, P + s + 5:] = m.mask_id
    cfg = Bd.Engine.cfg_struct(G, s, 0.5, bias=(m.eos_id, s + 9, 3.0))

    def step(tokens):
        tokens = tokens.clone()
        state = torch.tensor([[1, 2, 0]] * tokens.shape[0], dtype=torch.int32, device="cuda")
        out = Bd.Engine(m, weights, tokens.shape[0], P + G).denoise_step(tokens, P, state, flt, cfg, want_logits=True)
        return dict(out, tokens=tokens)
    many = step(X)
    for b in range(B):
        one = step(X[b:b + 1])
        for k in one:
            assert torch.equal(one[k][0], many[k][b]), (b, k)
