"""Tile edges of the many-row bf16 GEMMs: forwards of two-layer models (the last layer may work on the wanted rows alone,
the first one works on all of them) whose widths and row counts make the tile chooser take each of its tiles for each
product, with the row counts just below, at and above a tile, K from one 64-deep stage (fewer than the ring holds) to odd
numbers of them, output columns that no tile divides, and the LM head on 65, 128, 129 and 256 rows.  Same bound as the
other bf16 forwards: 2e-2 of the largest logit."""
import numpy as np
import pytest
import torch

from paper_2509_25188_amd import binding as Bd
from paper_2509_25188_amd import synth
from tests import parity as Pz

pytestmark = pytest.mark.gpu

CASES = [
    # (d, H, Dh, F, V, B, T, head rows); the first layer's tiles are 128 x 64 where no other is named
    (64, 1, 64, 64, 300, 1, 65, 65),          # one stage of K, one tile, a row more than the few-row path
    (64, 1, 64, 128, 257, 1, 128, 128),       # K of one and two stages
    (192, 3, 64, 320, 385, 1, 129, 129),      # three and five stages; LM head 256 x 256 with one row in its second half
    (256, 2, 128, 320, 500, 2, 128, 64),      # 256 rows in two sequences
    (256, 4, 64, 448, 640, 1, 257, 256),      # one row in the second 256-row tile
    (256, 2, 128, 12288, 300, 1, 700, 32),    # gate/up 256 x 192 tiles, down K = 12288 in four ranges
    (256, 2, 128, 12288, 300, 3, 401, 32),    # gate/up 256 x 256 tiles, 1203 rows over three sequences
    (128, 2, 64, 8320, 300, 1, 129, 32),      # gate/up 128 x 192, ragged columns
    (128, 2, 64, 12352, 300, 1, 255, 200),    # gate/up 256 x 128, a row short of the tile; more than half of the rows wanted
    (128, 2, 64, 8320, 300, 1, 257, 32),      # gate/up 256 x 192, ragged columns, a row more than the tile
    (128, 2, 64, 12352, 300, 1, 257, 129),    # gate/up 256 x 256, ragged columns
    (1344, 21, 64, 128, 300, 1, 513, 32),     # Q/K/V 128 x 128, ragged columns
    (2048, 16, 128, 128, 300, 1, 769, 32),    # Q/K/V 128 x 192; output projection 256 x 128, four ranges
    (832, 13, 64, 128, 300, 3, 853, 32),      # Q/K/V 256 x 128, ragged columns, 2559 rows (a row short of the tile)
    (1664, 13, 128, 128, 300, 5, 461, 16),    # Q/K/V 256 x 256, ragged columns, 2305 rows; output projection 256 x 192, two ranges
    (320, 5, 64, 2048, 300, 3, 512, 32),      # gate/up 256 x 128; down 128 x 128, four ranges, ragged columns
    (832, 13, 64, 2048, 300, 5, 461, 16),     # gate/up 256 x 192; down 256 x 192, four ranges, ragged columns
    (1216, 19, 64, 2048, 300, 5, 461, 16),    # Q/K/V 256 x 192; down 256 x 256, four ranges, ragged columns
    (1344, 21, 64, 2048, 300, 3, 853, 16),    # down 256 x 128, a workgroup walking the four ranges, ragged columns
    (512, 4, 128, 8192, 300, 2, 513, 200),    # 1026 rows, gate/up 256 x 192, down 128 x 128; head rows of two sequences in slabs
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_tile_edges(case):
    d, H, Dh, F, V, B, T, rows = CASES[case]
    m = synth.ModelShape(2, d, H, Dh, F, V, V - 1, V - 2, dtype="bf16")
    weights = synth.make_weights(m, 240 + case, "cpu")
    ora = Pz.oracle_model(m, weights, gemm_input="bf16")
    eng = Bd.Engine(m, Pz.to_dev(weights), B, T)
    X = synth.make_prompt(260 + case, B, T, V - 2, "cpu")
    got = eng.forward(X.cuda(), T - rows, rows)
    again = eng.forward(X.cuda(), T - rows, rows)
    assert torch.equal(got, again)
    got = got.cpu().numpy()
    for b in sorted({0, B // 2, B - 1}):
        ref = ora.forward(X[b].numpy())[T - rows:]
        assert Pz.rel_err(got[b], ref) < 2e-2, b


def test_rows_are_the_same_bits_in_every_tile():
    # the same 300 rows alone (128- or 256-row tiles, a workgroup per K range) and as the first of nine sequences
    # (larger tiles, K ranges walked by one workgroup): row by row the same sums in the same order
    m = synth.ModelShape(1, 2048, 16, 128, 4096, 300, 299, 298, dtype="bf16")
    eng = Bd.Engine(m, synth.make_weights(m, 3, "cuda"), 9, 300)
    X = synth.make_prompt(5, 9, 300, 298, "cuda")
    many = eng.forward(X, 0, 200)
    for b in (0, 4, 8):
        alone = eng.forward(X[b:b + 1].contiguous(), 0, 200)
        assert torch.equal(alone[0], many[b]), b


@pytest.mark.parametrize("B,row,rows", [(1, 100, 40), (1, 0, 130), (3, 31, 64), (3, 177, 110)])
def test_wanted_rows_are_the_same_bits_as_all_rows(B, row, rows):
    # logits of some rows (the last layer works on those alone behind its keys and values: few-row and tile kernels,
    # query tiles without a wanted row skipped) against the same rows of a forward that returns them all
    m = synth.ModelShape(2, 2048, 16, 128, 4096, 300, 299, 298, dtype="bf16")
    eng = Bd.Engine(m, synth.make_weights(m, 3, "cuda"), B, 300)
    X = synth.make_prompt(6, B, 300, 298, "cuda")
    every = eng.forward(X, 0, 300)
    some = eng.forward(X, row, rows)
    assert torch.equal(some, every[:, row:row + rows])


@pytest.mark.parametrize("d,F,B,T,row,rows", [
    (2048, 4096, 1, 100, 31, 40), (2048, 4096, 1, 256, 0, 128), (2048, 4096, 2, 120, 7, 50), (1024, 2816, 3, 77, 40, 36),
    (4096, 12288, 1, 100, 60, 32), (4096, 12288, 2, 128, 3, 64),
])
def test_wanted_rows_of_a_short_pass_are_the_same_bits_as_all_rows(d, F, B, T, row, rows):
    # the same for passes of 65 to 256 rows, whose projections choose their K ranges by the row count: the last layer's wanted
    # rows sum in the ranges of the pass that they belong to
    m = synth.ModelShape(2, d, d // 128, 128, F, 300, 299, 298, dtype="bf16")
    eng = Bd.Engine(m, synth.make_weights(m, 3, "cuda"), B, T)
    X = synth.make_prompt(6, B, T, 298, "cuda")
    every = eng.forward(X, 0, T)
    some = eng.forward(X, row, rows)
    assert torch.equal(some, every[:, row:row + rows])
