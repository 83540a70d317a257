"""The buffer for split-K partials holds those of every pass an engine may run, not only of a pass as large as the engine:
fewer rows may sum in more ranges.  The planners and the size carved by the workspace layout are read from the library."""
import ctypes as C

import pytest
import torch

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth
from tests import parity as Pz

FEW = 64          # rows up to which a pass takes the few-row kernels
ROWS = 700        # engines of up to this many rows
FFN = (1024, 2048, 2816, 6144, 6656, 12288)
WIDTHS = (64, 576, 1024, 1088, 1152, 1216, 1344, 1536, 2048, 2752, 3072, 4096)


def planners():
    lib = Bd.lib()
    wide, few, ranges, size = (getattr(lib, n) for n in ("_ZN4l2pd11wide_splitsEiiii", "_ZN4l2pd13skinny_splitsEii",
                                                         "_ZN4l2pd8k_rangesEiii", "_ZN4l2pd14partial_floatsExii"))
    size.restype, size.argtypes = C.c_size_t, [C.c_longlong, C.c_int, C.c_int]
    return wide, few, ranges, size


def gate_up_ranges(F, d):
    """Whether gate/up of few rows writes partial sums: the third of its ways."""
    return Bd.lib()._ZN4l2pd16few_rows_gate_upEiib(F, d, True) == 2


def few_rows_need(few, d, F):
    """Columns times ranges of the widest set of partial sums that a pass of up to 64 rows writes."""
    sums = [(d, d), (d, F)] + ([(2 * F, d)] if gate_up_ranges(F, d) else [])
    return max(few(n, k) * n for n, k in sums)


@pytest.mark.parametrize("d", WIDTHS)
def test_every_pass_fits(d):
    wide, few, ranges, size = planners()
    for F in FFN:
        most = 0
        for M in range(1, ROWS + 1):
            if M <= FEW:
                need = few_rows_need(few, d, F) * M
            else:
                tail = M // 2        # the most wanted rows that the last layer's projections work on alone
                need = max(wide(M, d, k, M) * M * d for k in (d, F))
                need = max(need, *(ranges(M, d, k) * min(tail, FEW) * d for k in (d, F)))
                if tail > FEW:
                    need = max(need, *(wide(tail, d, k, M) * tail * d for k in (d, F)))
            most = max(most, need)
            assert size(M, d, F) >= most, (d, F, M)


@pytest.mark.parametrize("d", WIDTHS + (1600, 2816))
def test_small_engines_hold_no_more_than_their_sums(d):
    wide, few, ranges, size = planners()
    for F in FFN + (64, 1984):
        for rows in (2, 32, FEW):
            assert size(rows, d, F) == few_rows_need(few, d, F) * rows, (F, rows)


@pytest.mark.gpu
@pytest.mark.parametrize("d,F", [(1088, 2048), (576, 6144)])
def test_small_pass_of_a_larger_engine_matches_oracle(d, F):
    # 192 rows sum the down projection in twice as many ranges as 256
    m = synth.ModelShape(2, d, d // 64, 64, F, 300, 299, 298, dtype="bf16")
    weights = synth.make_weights(m, 710, "cpu")
    eng = Bd.Engine(m, Pz.to_dev(weights), 1, 256)
    X = synth.make_prompt(711, 1, 192, 298, "cpu")
    got = eng.forward(X.cuda())
    assert torch.equal(got, Bd.Engine(m, Pz.to_dev(weights), 1, 192).forward(X.cuda()))
    assert Pz.rel_err(got[0].cpu().numpy(), Pz.oracle_model(m, weights, gemm_input="bf16").forward(X[0].numpy())) < 2e-2
