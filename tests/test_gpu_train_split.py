"""Filter training with its rows dealt to workgroups (l2pd_filter_train_split) against the oracle and against the
one-workgroup entry point: ragged last workgroups, several chunks of rows in one workgroup, one launch an epoch and two,
widths that are no multiple of 16, one to four layers."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import l2pd_oracle as O
from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth
from tests import parity as Pz

pytestmark = pytest.mark.gpu


def train(flt, conf, label, epochs, split):
    lib = Bd.lib()
    f = Bd._filter_struct(flt)
    n = conf.shape[0]
    need = lib.l2pd_filter_train_workspace_bytes(C.byref(f), n)
    n_params = sum(t.numel() for t in flt.values())
    opt = torch.full((2 * n_params,), float("nan"), device="cuda")
    loss = torch.full((epochs,), float("nan"), device="cuda")
    work = torch.full((max(need, 4) // 4,), float("nan"), device="cuda")     # never read before it is written
    tc = Bd.TrainCfg(1e-3, 0.9, 0.999, 1e-8, 0.01, epochs)
    rc = lib.l2pd_filter_train_split(C.byref(f), conf.data_ptr(), label.data_ptr(), n, C.byref(tc), opt.data_ptr(),
                                     loss.data_ptr(), work.data_ptr() if split else None, need if split else 0,
                                     torch.cuda.current_stream().cuda_stream)
    assert rc == Bd.L2PD_OK
    return need, opt, loss


# width, hidden, layers, rows; workgroups (1: not split) and launches an epoch that the plan takes.  The last has several chunks
# of rows in a workgroup.
SHAPES = [(32, 32, 2, 241, 16, 1), (32, 32, 2, 129, 9, 1), (64, 128, 2, 4096, 128, 2), (64, 128, 2, 17, 1, 0),
          (24, 40, 3, 333, 21, 2), (20, 1, 1, 1001, 21, 1), (48, 48, 4, 2049, 65, 2), (1, 1, 2, 5000, 53, 1),
          (32, 32, 2, 20011, 126, 2), (128, 64, 2, 3001, 94, 2), (64, 128, 2, 16387, 114, 2)]


def workspace_bytes(s, h, L, groups, launches):
    """What such a plan asks for: two states of three images (parameters padded to 16, moments), and a partial gradient with
    the losses of 16 wavefronts per workgroup, twice where one launch both applies and writes them."""
    if groups == 1:
        return 0
    widths = [(x + 15) // 16 * 16 for x in [s] + [h] * (L - 1) + [s]]
    image = sum(a * b for a, b in zip(widths, widths[1:])) + sum(widths[1:])
    assert (groups * (image + 16) <= 1 << 16) == (launches == 1)      # partial gradients that every workgroup can read
    return 4 * (6 * image + (2 if launches == 1 else 1) * groups * (image + 16))


@pytest.mark.parametrize("s,h,L,n,groups,launches", SHAPES)
def test_rows_over_workgroups_match_oracle_and_one_workgroup(s, h, L, n, groups, launches):
    r = np.random.default_rng(91)
    Cn = r.uniform(size=(n, s)).astype(np.float32)
    Yn = (r.uniform(size=(n, s)) < 0.2 + 0.6 * Cn).astype(np.float32)
    flt = synth.make_filter(92, s, h, "cpu", n_layers=L)
    Cd, Yd = torch.tensor(Cn).cuda(), torch.tensor(Yn).cuda()
    epochs = 4
    one = {k: v.clone().cuda() for k, v in flt.items()}
    many = {k: v.clone().cuda() for k, v in flt.items()}
    _, opt1, loss1 = train(one, Cd, Yd, epochs, False)
    need, opt, loss = train(many, Cd, Yd, epochs, True)
    again = {k: v.clone().cuda() for k, v in flt.items()}
    train(again, Cd, Yd, epochs, True)
    assert groups <= (n + 15) // 16 and need == workspace_bytes(s, h, L, groups, launches)
    ref, ref_losses = O.train_filter(Pz.np_filter(flt), Cn, Yn, epochs, lr=1e-3)
    np.testing.assert_allclose(loss.cpu().numpy(), ref_losses, rtol=1e-5, atol=1e-7)
    np.testing.assert_allclose(loss1.cpu().numpy(), ref_losses, rtol=1e-5, atol=1e-7)
    for k in ref:
        assert torch.equal(again[k], many[k]), k
        # four updates of at most 1e-3 each; where a gradient entry is rounding noise its sign is free
        d = np.abs(many[k].cpu().numpy() - ref[k])
        assert d.max() < 8.5e-3 and np.mean(d < 1e-4) > 0.995, (k, d.max())
    # moments: gradients to the rounding of their sums, relative to the largest entry
    N = opt.numel() // 2
    for a, b in ((opt[:N], opt1[:N]), (opt[N:], opt1[N:])):
        assert torch.isfinite(a).all()
        assert float((a - b).abs().max()) <= 2e-4 * float(b.abs().max())


def test_workspace_is_checked_before_any_launch():
    lib = Bd.lib()
    flt = {k: v.cuda() for k, v in synth.make_filter(93, 32, 32, "cpu").items()}
    f = Bd._filter_struct(flt)
    rows = torch.zeros((500, 32), device="cuda")
    need = lib.l2pd_filter_train_workspace_bytes(C.byref(f), 500)
    assert need > 0
    opt, work = torch.zeros(2 * 2112, device="cuda"), torch.zeros(need // 4 + 64, device="cuda")
    tc = Bd.TrainCfg(1e-3, 0.9, 0.999, 1e-8, 0.01, 1)
    w1 = flt["w1"].clone()

    def call(ptr, nbytes):
        return lib.l2pd_filter_train_split(C.byref(f), rows.data_ptr(), rows.data_ptr(), 500, C.byref(tc),
                                           opt.data_ptr(), None, ptr, nbytes, torch.cuda.current_stream().cuda_stream)
    assert call(work.data_ptr(), need - 4) == Bd.L2PD_ENOMEM
    assert call(work.data_ptr() + 4, need) == Bd.L2PD_EINVAL
    torch.cuda.synchronize()
    assert torch.equal(flt["w1"], w1)


@pytest.mark.parametrize("s,h,n", [(32, 32, 241), (64, 128, 700)])     # one launch an epoch, and two
def test_captured_training_equals_the_eager_one_on_every_replay(s, h, n):
    r = np.random.default_rng(94)
    conf = torch.tensor(r.uniform(size=(n, s)).astype(np.float32)).cuda()
    label = (conf > 0.5).float()
    first = {k: v.cuda() for k, v in synth.make_filter(95, s, h, "cpu").items()}
    flt = {k: v.clone() for k, v in first.items()}
    epochs = 40
    want = Bd.train_filter(flt, conf, label, epochs, static_scratch=True).clone()      # (looks the array's address up)
    trained = {k: v.clone() for k, v in flt.items()}
    losses = torch.empty(epochs, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        Bd.train_filter(flt, conf, label, epochs, losses=losses, static_scratch=True)
    for _ in range(4):
        for k in flt:
            flt[k].copy_(first[k])
        losses.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(losses, want)
        for k in flt:
            assert torch.equal(flt[k], trained[k]), k
        # eager work in between, in the same array
        other = {k: v.clone() for k, v in first.items()}
        Bd.train_filter(other, conf[:150], label[:150], 3, static_scratch=True)
