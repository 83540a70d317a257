"""Block-only steps of up to 64 rows: the projections sum in the same K ranges however many sequences share the launch, so that
(below 512 keys, from where on few workgroups deal the keys among them) a sequence's logits are those of its own single run,
bit for bit, in the tiles of 32 rows and of 64.  The store is rebuilt from passes above 256 rows, which sum alike too."""
import pytest
import torch

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # (d, head size, FFN, batch, block, prompt): rows 32 and 64, 16 and 48 and 64, 24 and 48, 20 and 60
    (2048, 128, 8192, 2, 32, 230), (4096, 128, 12288, 2, 32, 230), (4096, 128, 4096, 3, 16, 250), (2048, 64, 8192, 4, 16, 250),
    (1024, 64, 2816, 2, 24, 250), (2048, 128, 2816, 3, 20, 260),
]


@pytest.mark.parametrize("d,Dh,F,B,s,P", CASES)
@pytest.mark.parametrize("prefix", [False, True])
def test_logits_of_a_sequence_do_not_depend_on_the_batch(d, Dh, F, B, s, P, prefix):
    m = synth.ModelShape(2, d, d // Dh, Dh, F, 300, 299, 298, dtype="bf16")
    weights = synth.make_weights(m, 840, "cuda")
    flt = synth.make_filter(841, s, 32, "cuda")
    G = 3 * s
    X = synth.make_prompt(842, B, P + G, 298, "cuda")
    X[:, P + s + 3:] = m.mask_id

    def step(tokens):
        tokens = tokens.clone()
        n = tokens.shape[0]
        cfg = Bd.Engine.cfg_struct(G, s, 0.9, prefix_cache=prefix, dual_cache=not prefix)
        eng = Bd.Engine(m, weights, n, P + G, True)
        state = torch.tensor([[1, 0, 0]] * n, dtype=torch.int32, device="cuda")
        return eng.denoise_step(tokens, P, state, flt, cfg, want_logits=True)["logits"]
    many = step(X)
    assert torch.equal(many, step(X))
    for b in range(B):
        assert torch.equal(step(X[b:b + 1])[0], many[b]), b
