"""A weight gradient and an x W^T in one launch (ecospa_gemm_pair) against the same two one after the other, bit for bit: every pair of tile
shapes that is built, ragged sizes, K split and not, with and without column sums; and buffers that make the order matter."""
import ctypes as C

import pytest
import torch

from paper_2511_11641_amd import binding as B
from util import GemmDesc

pytestmark = pytest.mark.gpu
ONE, PAIR, ROWS = "_Z11ecospa_gemmP10ecospa_ctxRK8GemmDesc", "_Z16ecospa_gemm_pairP10ecospa_ctxRK8GemmDescS3_", "_Z23ecospa_gemm_colsum_rowsRK8GemmDesc"


@pytest.fixture(scope="module")
def ctx():
    return B.Context("cuda:0")


def _desc(M, N, K, a, b, tt, tile, splits=1, partial=None):
    c = torch.full((M, N), 7.0, device="cuda").bfloat16()
    g = GemmDesc(B.BF16, M, N, K, a.data_ptr(), a.stride(0), int(tt), b.data_ptr(), b.stride(0), int(tt), tile, splits,
                 partial.data_ptr() if partial is not None else None, int(splits > 1))
    g.epi.c, g.epi.ldc = c.data_ptr(), N
    return g, c


@pytest.mark.parametrize("w_tile", [39, 38, 37, 34])                 # 64, 128, 192, 256 x 128
@pytest.mark.parametrize("x_tile", [34, 35, 37, 38])                 # 256 x 128, 192 x 192, 192 x 128, 128 x 128
@pytest.mark.parametrize("T,d,n,splits,sums", [(1379, 264, 392, 1, True), (1379, 392, 264, 3, False), (63, 136, 520, 1, False), (4191, 200, 72, 4, True)])
def test_one_launch_gives_what_two_give(ctx, w_tile, x_tile, T, d, n, splits, sums):
    gen = torch.Generator(device="cuda").manual_seed(81)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen).bfloat16()
    dh, x, wt = rnd(T, n), rnd(T, d), rnd(d, n)
    out = []
    for pair in (False, True):
        part = torch.full((splits, n, d), 7.0, device="cuda")
        w, dw = _desc(n, d, T, dh, x, True, w_tile, splits, part)
        rows = getattr(ctx.lib, ROWS)(C.byref(w))
        cs = torch.full((rows, n), 7.0, device="cuda")
        if sums:
            w.colsum = cs.data_ptr()
        g, dx = _desc(T, d, n, dh, wt, False, x_tile)
        if pair:
            assert getattr(ctx.lib, PAIR)(ctx.h, C.byref(w), C.byref(g)) == B.OK
        else:
            assert getattr(ctx.lib, ONE)(ctx.h, C.byref(w)) == B.OK and getattr(ctx.lib, ONE)(ctx.h, C.byref(g)) == B.OK
        out.append((dw, part, cs, dx))
    for one, two in zip(*out):
        assert torch.equal(one, two)
    assert not bool((out[1][3] == 7.0).all())


def test_an_input_that_the_other_overwrites_is_read_first(ctx):
    gen = torch.Generator(device="cuda").manual_seed(82)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen).bfloat16()
    dh, x, wt = rnd(1379, 392), rnd(1379, 264), rnd(264, 392)
    want = dh.float().t() @ x.float()
    w, dw = _desc(392, 264, 1379, dh, x, True, 0)
    g, _ = _desc(1379, 264, 392, dh, wt, False, 0)
    g.epi.c = x.data_ptr()                    # the input gradient goes where the weight gradient's input is
    assert getattr(ctx.lib, PAIR)(ctx.h, C.byref(w), C.byref(g)) == B.OK
    # bf16 rounding of the result: 2^-9 of each element at most
    assert float((dw.float() - want).norm() / want.norm()) < 2 ** -8
