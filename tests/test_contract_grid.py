"""The grid of a contraction launch (csrc/gemm.hip: gemm_ring_grid), asked of the host function that the launches go by; the kernels' decoding of a
workgroup's number is written out here in plain integers."""
import ctypes as C
import random

import pytest

from paper_2511_11641_amd import binding as B

SHAPES = [(256, 256), (192, 256), (256, 192), (128, 256), (256, 128), (192, 192), (128, 192), (192, 128), (128, 128), (64, 128), (128, 64), (64, 64),
          (32, 16), (32, 32), (64, 16), (64, 32)]


class RingGrid(C.Structure):
    _fields_ = [(n, C.c_int) for n in "tiles_n k_chunk per more tiles group band last_band last_rows".split()] + [
        (n, C.c_uint) for n in "tiles_inv band_inv group_inv last_inv".split()]


def _grid(M, N, bm, bn, splits=1):
    f = B.load()._Z14gemm_ring_gridiiiiii
    f.restype = RingGrid
    return f(M, N, bm, bn, splits, 64)


def _div(a, d, inv):
    """ring_div of csrc/gemm_ring.h: the high half of a product, one correction."""
    q = (a * inv) >> 32
    r = a - q * d
    return (q + 1, r - d) if r >= d else (q, r)


def _tile(g, block, splits):
    xcd = block & 7
    i = xcd * g.per + min(xcd, g.more) + (block >> 3)
    z, i = _div(i, g.tiles, g.tiles_inv) if splits > 1 else (0, i)
    band, i = _div(i, g.band, g.band_inv)
    last = band == g.last_band
    col, row = _div(i, g.last_rows if last else g.group, g.last_inv if last else g.group_inv)
    return z, band * g.group + row, col


@pytest.mark.parametrize("seed", range(4))
def test_every_tile_of_every_split_has_one_workgroup(seed):
    rng = random.Random(seed)
    for _ in range(60):
        bm, bn = rng.choice(SHAPES)
        tm, tn, splits = rng.choice((1, 2, 3, 5, 17, 64, 129)), rng.choice((1, 2, 7, 8, 31, 50)), rng.choice((1, 1, 2, 3, 8))
        g = _grid(tm * bm - rng.randrange(bm), tn * bn - rng.randrange(bn), bm, bn, splits)
        assert (g.tiles, g.tiles_n, g.per * 8 + g.more) == (tm * tn, tn, tm * tn * splits)
        seen = {_tile(g, b, splits) for b in range(tm * tn * splits)}
        assert seen == {(z, r, c) for z in range(splits) for r in range(tm) for c in range(tn)}


def _rows_fetched(tm, tn, bm, bn, height):
    """Operand rows that an XCD's tiles of a launch of one round read, mean of the eight."""
    total = 0
    for xcd in range(8):
        per, more = divmod(tm * tn, 8)
        first = xcd * per + min(xcd, more)
        rows, cols = set(), set()
        for i in range(first, first + per + (xcd < more)):
            band, j = divmod(i, height * tn)
            h = min(height, tm - band * height)
            rows.add(band * height + j % h)
            cols.add(j // h)
        total += len(rows) * bm + len(cols) * bn
    return total / 8


@pytest.mark.parametrize("bm,bn", SHAPES)
def test_few_tile_rows_are_not_cut_into_bands_that_fetch_more(bm, bn):
    """Up to eight tile rows, half a round and more: the height taken is at most an eighth above the best, where ranges of an XCD that straddle two
    bands or end inside a column are counted too (which the rule does not; five tile rows in bands of three and two would be up to 1.35)."""
    for tm in range(1, 9):
        for tn in range(max(1, 128 // tm), 256 // tm + 1):
            got = _rows_fetched(tm, tn, bm, bn, _grid(tm * bm, tn * bn, bm, bn).group)
            assert got <= 1.125 * min(_rows_fetched(tm, tn, bm, bn, h) for h in range(1, tm + 1)), (tm, tn)


def test_several_rounds_keep_bands_of_a_fixed_height():
    for (bm, bn), rows in (((256, 256), 4), ((192, 256), 4), ((128, 64), 8), ((64, 64), 16)):
        assert _grid(64 * bm, 7 * bn, bm, bn).group == rows
        assert _grid(3 * bm, 200 * bn, bm, bn).group == 3
