"""A weight gradient and an x W^T in one launch (ecospa_gemm_pair) against the same two one after the other, bit for bit: every pair of tile
shapes that is built, ragged sizes, K split and not, with and without column sums; and buffers that make the order matter."""
import ctypes as C

import pytest
import torch

from paper_2511_11641_amd import binding as B
from util import GemmDesc

pytestmark = pytest.mark.gpu
ONE, PAIR, ROWS = "_Z11ecospa_gemmP10ecospa_ctxRK8GemmDesc", "_Z16ecospa_gemm_pairP10ecospa_ctxRK8GemmDescS3_i", "_Z23ecospa_gemm_colsum_rowsRK8GemmDesc"

PAIR_ROUTE = "_Z22ecospa_gemm_pair_routeRK8GemmDescS1_PiS2_"      # 0: two launches, 1: one of bf16, 2: one of fp32


def _route(ctx, w, x):
    ws, xs = C.c_int(), C.c_int()
    return getattr(ctx.lib, PAIR_ROUTE)(C.byref(w), C.byref(x), C.byref(ws), C.byref(xs)), ws.value, xs.value


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
            # tile codes 30 .. 41 in the order of the shapes
            assert _route(ctx, w, g) == (1, w_tile - 30, x_tile - 30)
            assert getattr(ctx.lib, PAIR)(ctx.h, C.byref(w), C.byref(g), 0) == B.OK
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
    w, dw = _desc(392, 264, 1379, dh, x, True, 39)
    g, _ = _desc(1379, 264, 392, dh, wt, False, 38)
    assert _route(ctx, w, g)[0] == 1
    g.epi.c = x.data_ptr()                    # the input gradient goes where the weight gradient's input is
    assert _route(ctx, w, g)[0] == 0
    assert getattr(ctx.lib, PAIR)(ctx.h, C.byref(w), C.byref(g), 0) == B.OK
    # bf16 rounding of the result: 2^-9 of each element at most
    assert float((dw.float() - want).norm() / want.norm()) < 2 ** -8


@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("T,d,n", [(512, 256, 512), (61, 40, 72), (1, 8, 33), (701, 96, 1500)])
def test_fp32_pair_and_column_sums(ctx, T, d, n, tb):
    """fp32: the same two contractions, x with W stored either way, and the column sums of the weight gradient's first operand."""
    gen = torch.Generator(device="cuda").manual_seed(83)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    dh, x, wm = rnd(T, n), rnd(T, d), rnd(*((n, d) if tb else (d, n)))
    dw, dx, cs = (torch.full(s, 7.0, device="cuda") for s in ((n, d), (T, d), (n,)))
    w = GemmDesc(B.F32, n, d, T, dh.data_ptr(), n, 1, x.data_ptr(), d, 1, 0, 1, None)
    g = GemmDesc(B.F32, T, d, n, dh.data_ptr(), n, 0, wm.data_ptr(), wm.stride(0), tb, 0, 1, None)
    w.epi.c, w.epi.ldc, w.colsum, g.epi.c, g.epi.ldc = dw.data_ptr(), d, cs.data_ptr(), dx.data_ptr(), d
    assert _route(ctx, w, g)[0] == 2
    assert getattr(ctx.lib, PAIR)(ctx.h, C.byref(w), C.byref(g), 0) == B.OK
    for got, want in ((dw, dh.double().t() @ x.double()), (dx, dh.double() @ (wm.double() if tb else wm.double().t())), (cs, dh.double().sum(0))):
        assert float((got - want).norm() / want.norm()) < 2e-6      # chains of at most 256 fp32 additions


@pytest.mark.parametrize("T,d,n", [(512, 256, 512), (61, 40, 72), (70, 1024, 2048)])      # K shared out over the wavefronts; 64 x 64 tiles
def test_fp32_column_sums_of_infinities(ctx, T, d, n):
    """One infinite gradient, an overflow, both signs, not a number: as a plain sum has them, and the other columns as without."""
    gen = torch.Generator(device="cuda").manual_seed(84)
    dh, x, dw = (torch.randn(s, device="cuda", generator=gen) for s in ((T, n), (T, d), (n, d)))
    sums = []
    for special in (False, True):
        if special:
            dh[3, 5], dh[T - 1, 7], dh[0, 9] = float("inf"), float("-inf"), float("nan")
            dh[4, 11], dh[T - 2, 11] = float("inf"), float("-inf")
            dh[1, 13], dh[2, 13] = 3e38, 3e38
        cs = torch.full((n,), 7.0, device="cuda")
        w = GemmDesc(B.F32, n, d, T, dh.data_ptr(), n, 1, x.data_ptr(), d, 1, 0, 1, None)
        w.epi.c, w.epi.ldc, w.colsum = dw.data_ptr(), d, cs.data_ptr()
        assert getattr(ctx.lib, ONE)(ctx.h, C.byref(w)) == B.OK
        sums.append(cs)
    plain, cs = sums
    assert float(cs[5]) == float("inf") and float(cs[7]) == float("-inf") and float(cs[13]) == float("inf")
    assert bool(torch.isnan(cs[[9, 11]]).all())
    rest = torch.ones(n, dtype=torch.bool, device="cuda")
    rest[[5, 7, 9, 11, 13]] = False
    assert torch.equal(cs[rest], plain[rest])
