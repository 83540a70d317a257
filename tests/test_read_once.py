"""Which launches load weights with the hint for data used once: one row tile, or row tiles that read every panel together.  The rule is
read from the library; where the tiles of a launch land is worked out here (workgroups go to the eight XCDs in turn)."""
import ctypes as C

import pytest

from paper_2509_25188_amd import binding as Bd

TILES = ((256, 256), (256, 192), (256, 128), (128, 192), (128, 128), (128, 64), (64, 128), (64, 64), (64, 32), (32, 128), (32, 32))
COLUMNS = (1024, 3072, 4608, 8192, 10752, 12288, 15360, 24576, 126464)


def read_once(M, N, splits, bm, bn):
    f = Bd.lib()._ZN4l2pd9read_onceEiiiii
    f.restype = C.c_bool
    return f(M, N, splits, bm, bn)


def panel_xcds(tiles_m, tiles_n, splits):
    """The XCDs of every panel's row tiles: ids dealt to an XCD are consecutive, the row tiles of a panel too."""
    total = tiles_m * tiles_n * splits
    per_xcd = (total + 7) // 8
    return [{v // per_xcd for v in range(p * tiles_m, (p + 1) * tiles_m)} for p in range(tiles_n * splits)]


@pytest.mark.parametrize("bm,bn", TILES)
def test_hint_only_where_a_panel_is_read_together(bm, bn):
    for N in COLUMNS:
        for splits in (1, 2, 4):
            for M in range(1, 600):
                tiles_m = -(-M // bm)
                got = read_once(M, N, splits, bm, bn)
                if M > 512:
                    assert not got
                elif tiles_m == 1:
                    assert got
                elif got:
                    last = M - (tiles_m - 1) * bm
                    assert min(bm, bn) >= 128 and (bm == 256 or 4 * last >= 3 * bm), (M, N)
                    assert all(len(x) == 1 for x in panel_xcds(tiles_m, -(-N // bn), splits)), (M, N)


def test_both_sides_of_the_line():
    assert all(read_once(M, 12288, 1, 128, 128) for M in (224, 256))
    assert not any(read_once(M, 12288, 1, 128, 128) for M in (129, 192, 257))
    assert not any(read_once(M, 10752, 1, 128, 128) for M in (224, 256))       # 21 tiles to an XCD
    assert not any(read_once(M, 10752, 1, 64, 64) for M in (176, 192))
    assert all(read_once(M, 24576, 1, 256, 192) for M in (257, 512)) and read_once(512, 12288, 1, 128, 192)
    assert not any(read_once(M, 27648, 1, 256, 256) for M in (257, 512))       # 27 tiles to an XCD
