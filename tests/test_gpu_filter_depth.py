"""GPU parity for the filter-depth variants of Table 3 (one, two and four layers): decoding with each,
teacher-forced and free-running, and training each, against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import l2pd_oracle as O
from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth
from tests import parity as Pz
from tests.test_gpu_parity import build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_layers,hidden", [(1, 64), (2, 64), (4, 64), (4, 48), (3, 200)])
def test_decode_with_filters_of_each_depth_fp32(n_layers, hidden):
    w = synth.WORKLOADS["tiny"]
    eng, ora, _, prompt = build(w, lm_head_scale=25.0)
    flt = synth.make_filter(77, w.block_len, hidden, "cpu", n_layers=n_layers)
    assert len(flt) == 2 * n_layers
    trace = []
    resp, steps, dlen = Pz.oracle_generate(ora, prompt[0].numpy(), w, Pz.np_filter(flt), trace)
    fdev = {k: v.cuda() for k, v in flt.items()}
    cfg = Pz.cfg_for(w)
    rep = Pz.StepReport()
    forced = Pz.teacher_forced(eng, [trace], w.prompt_len, cfg, fdev, w.model, w.threshold, rep)
    print(f"{n_layers}-layer filter (hidden {hidden}): {rep}; oracle steps {steps}")
    assert rep.max_p_err < 1e-4
    assert rep.exempt_tokens == 0 and rep.exempt_decisions <= 1
    tok, st, dl = eng.generate(prompt.cuda(), fdev, cfg)
    Pz.check_generate(tok.cpu().numpy()[0], st[0], dl[0], trace, resp, steps, dlen, forced.first_exempt[0],
                      w.prompt_len, w.block_len, f"{n_layers}-layer filter")


def test_single_layer_filter_equals_two_layer_with_identity_first_layer():
    # the reduction the oracle is pinned with, on the device: same decisions, same trajectory
    w = synth.WORKLOADS["tiny"]
    eng, ora, _, prompt = build(w, lm_head_scale=25.0)
    s = w.block_len
    one = synth.make_filter(78, s, s, "cuda", n_layers=1)
    two = {"w1": torch.eye(s, device="cuda"), "b1": torch.zeros(s, device="cuda"), "w2": one["w1"], "b2": one["b1"]}
    cfg = Pz.cfg_for(w)
    a = eng.generate(prompt.cuda(), one, cfg)
    b = eng.generate(prompt.cuda(), two, cfg)
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("n_layers,s,h,n", [(1, 32, 32, 300), (4, 32, 32, 300), (4, 64, 64, 70), (3, 8, 5, 9),
                                            (1, 1, 1, 3)])
def test_training_filters_of_each_depth_matches_oracle(n_layers, s, h, n):
    r = np.random.default_rng(81)
    Cn = r.uniform(size=(n, s)).astype(np.float32)
    Yn = (r.uniform(size=(n, s)) < 0.2 + 0.6 * Cn).astype(np.float32)
    flt = synth.make_filter(82, s, h, "cpu", n_layers=n_layers)
    fdev = {k: v.clone().cuda() for k, v in flt.items()}
    Cd, Yd = torch.tensor(Cn).cuda(), torch.tensor(Yn).cuda()
    losses = Bd.train_filter(fdev, Cd, Yd, 20, lr=1e-3).cpu().numpy()
    ref, ref_losses = O.train_filter(Pz.np_filter(flt), Cn, Yn, 20, lr=1e-3)
    np.testing.assert_allclose(losses, ref_losses, rtol=1e-5, atol=1e-7)
    assert set(ref) == set(fdev)
    for k in ref:
        d = np.abs(fdev[k].cpu().numpy() - ref[k])
        assert np.mean(d < 1e-4) > 0.99 and d.max() < 2.5e-2, (k, d.max(), np.mean(d < 1e-4))
    # a longer run through losses and outputs (parameters may drift apart at equal loss once a ReLU
    # switches in one precision and not in the other)
    fdev = {k: v.clone().cuda() for k, v in flt.items()}
    losses = Bd.train_filter(fdev, Cd, Yd, 200, lr=3e-3).cpu().numpy()
    ref, ref_losses = O.train_filter(Pz.np_filter(flt), Cn, Yn, 200, lr=3e-3)
    print(f"{n_layers} layers, s {s}, hidden {h}, rows {n}: loss {losses[0]:.5f} -> {losses[-1]:.5f} "
          f"(oracle {ref_losses[0]:.5f} -> {ref_losses[-1]:.5f})")
    # The kernel trains in float32, the reference above in float64.  How far float32 arithmetic alone moves
    # the loss curve is measured on the oracle itself (same trainer in float32): the kernel may be that far
    # from the float64 curve (times two: two float32 evaluations differ from each other by up to twice what
    # each differs from the exact one), and never less than 1e-3 relative.  With more parameters than targets
    # (4 layers, 64 wide, 70 rows) the descent is ill-conditioned and the two oracle precisions themselves
    # part ways after some tens of steps; with enough rows they agree to 1e-4 and so must the kernel.
    _, ref32_losses = O.train_filter(Pz.np_filter(flt), Cn, Yn, 200, lr=3e-3, dtype=np.float32)
    spread = np.abs(ref32_losses - ref_losses)
    print(f"  float32 oracle vs float64 oracle: max loss distance {spread.max():.3e}; kernel vs float64 oracle "
          f"{np.abs(losses - ref_losses).max():.3e}")
    assert np.all(np.abs(losses - ref_losses) <= 2 * np.maximum.accumulate(spread) + 1e-3 * ref_losses + 1e-5)
    assert losses[-1] < losses[0]


def test_filters_too_large_for_the_training_kernel_are_refused():
    flt = synth.make_filter(83, 64, 128, "cuda", n_layers=4)      # 49,600 parameters
    C = torch.rand(10, 64, device="cuda")
    with pytest.raises(RuntimeError):
        Bd.train_filter(flt, C, (C > 0.5).float(), 2)


@pytest.mark.parametrize("n_layers,s,h,n", [
    (2, 16, 16, 16),      # one tile each way, one chunk without padding
    (2, 17, 33, 100),     # widths one over a tile; rows that fill part of the last tile
    (2, 32, 32, 256),     # the most rows that stay resident at this width
    (2, 32, 32, 257),     # one more: two chunks
    (3, 5, 7, 1),         # one row, everything padding
    (4, 48, 48, 130),     # hidden gradients in place of the outputs, two chunks
    (1, 128, 0, 70),      # single layer, five parameter tiles per wavefront
    (1, 140, 0, 40),      # more tiles than wavefronts hold: the scalar kernel
    (2, 16, 512, 30),     # likewise, two layers
])
def test_training_at_the_edges_of_the_kernels_tiles(n_layers, s, h, n):
    # fp32 sums over at most 256 rows and 512 inputs in another order than NumPy's float64: 20 steps stay within
    # 1e-5 of the loss and (where no ReLU switches) 1e-4 of a parameter, the bounds of the tests above
    r = np.random.default_rng(91)
    Cn = r.uniform(size=(n, s)).astype(np.float32)
    Yn = (r.uniform(size=(n, s)) < 0.2 + 0.6 * Cn).astype(np.float32)
    flt = synth.make_filter(92, s, h, "cpu", n_layers=n_layers)
    fdev = {k: v.clone().cuda() for k, v in flt.items()}
    losses = Bd.train_filter(fdev, torch.tensor(Cn).cuda(), torch.tensor(Yn).cuda(), 20, lr=1e-3).cpu().numpy()
    ref, ref_losses = O.train_filter(Pz.np_filter(flt), Cn, Yn, 20, lr=1e-3)
    np.testing.assert_allclose(losses, ref_losses, rtol=1e-5, atol=1e-7)
    for k in ref:
        d = np.abs(fdev[k].cpu().numpy() - ref[k])
        assert np.mean(d < 1e-4) > 0.99 and d.max() < 2.5e-2, (k, d.max(), np.mean(d < 1e-4))
