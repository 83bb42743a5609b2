"""The contraction kernel that shares K out over the wavefronts of a workgroup (csrc/gemm_share.h) against the kernel whose wavefronts share every
slab: every tile shape and epilogue, rows and columns off every tile, K from one part of a unit to more units than there are buffers, and
wavefronts without any."""
import ctypes as C

import pytest
import torch

from paper_2511_11641_amd import binding as B
from test_gpu_contract_flow import ACT, BIAS_ACT, DACT, DSWIGLU, ROPE, STORE, SWIGLU, _desc

pytestmark = pytest.mark.gpu
GEMM = "_Z11ecospa_gemmP10ecospa_ctxRK8GemmDesc"
RING_128 = 38          # tile code: 128 x 128 of the other kernel


@pytest.fixture(scope="module")
def ctx():
    return B.Context("cuda:0")


@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (33, 40, 56), (31, 72, 64), (65, 248, 520), (64, 96, 1608), (130, 24, 2048)])
@pytest.mark.parametrize("tile", [50, 51, 52, 53])
@pytest.mark.parametrize("kind,act,bias", [(STORE, 0, True), (STORE, 0, False), (BIAS_ACT, 0, True), (ACT, 0, False), (ACT, 1, True), (DACT, 0, True),
                                           (DSWIGLU, 0, True), (ROPE, 0, True), (SWIGLU, 0, True), (SWIGLU, 0, False)])
def test_shared_k_gives_what_shared_slabs_give(ctx, kind, act, bias, tile, M, N, K):
    if kind == ROPE and N < 144:
        N = 144          # four query and two key heads of 24
    gen = torch.Generator(device="cuda").manual_seed(81)
    g, c, c2, keep = _desc(kind, False, M, N, K, gen, bias, keep_c=bias or kind != SWIGLU)
    g.epi.act = (B.ACT_GELU_ERF, B.ACT_GELU_TANH)[act]
    _compare(ctx, g, c, c2, tile, M)
    del keep


def _compare(ctx, g, c, c2, tile, M, splits=1):
    """The launch of g on `tile`, K in `splits` parts, and on 128 x 128 tiles of the other kernel with K whole."""
    out = []
    parts = torch.full((splits * g.M * g.N + 64,), 7.0, device="cuda")
    for g.tile, g.splits, g.partial in ((tile, splits, parts.data_ptr() if splits > 1 else None), (RING_128, 1, None)):
        c.fill_(7.0)
        c2.fill_(7.0)
        assert getattr(ctx.lib, GEMM)(ctx.h, C.byref(g)) == B.OK
        out.append((c.clone(), c2.clone()))
    assert bool((parts[-64:] == 7).all()), "written beyond the partial sums"
    for x, y in zip(*out):
        assert bool((x[M:] == 7).all()) and bool((x[:, -8:] == 7).all()), "written beyond the matrix"
        # fp32 sums of up to 2048 products of size 1, in another order, differ by less than 2048^0.5 2^-24 4 = 1e-5; behind it bf16 rounds to a
        # neighbour at most (2^-7 of a value), of few values: a sum lies within 1e-5 of a rounding boundary 2^-8 apart
        assert bool(((x.float() - y.float()).abs() <= y.float().abs() * 2.0 ** -7 + 4e-5).all())
        assert float((x != y).float().mean()) < 0.03


@pytest.mark.parametrize("M,N,K", [(37, 40, 8), (37, 40, 56), (37, 72, 520), (37, 72, 1608)])
@pytest.mark.parametrize("tile", [50, 51, 52, 53, 38, 39, 40, 41])
def test_infinities_and_nan_stay_in_their_rows_and_columns(ctx, tile, M, N, K):
    """The k that fill the first unit up to 64 are zeroed behind the load, on both sides: nothing of them may meet an infinity or a NaN of the k that
    they repeat.  Every other output is as without them."""
    gen = torch.Generator(device="cuda").manual_seed(86)
    g, c, c2, (a, b, *keep) = _desc(STORE, False, M, N, K, gen)
    kv = (K - 1) % 64 + 1                        # k of the first unit
    for r, k, v in ((0, 0, float("inf")), (5, kv - 1, float("-inf")), (17, min(kv, K - 1), float("nan")), (36, K - 1, float("inf"))):
        a[r, k] = v
    for r, k, v in ((1, kv - 1, float("nan")), (8, 0, float("inf")), (N - 1, K - 1, float("-inf"))):
        b[r, k] = v
    g.tile = tile
    assert getattr(ctx.lib, GEMM)(ctx.h, C.byref(g)) == B.OK
    want = (a.double().cpu() @ b.double().cpu().T + keep[0].double().cpu()).cuda()
    got = c[:M, :N].double()
    assert bool((torch.isnan(got) == torch.isnan(want)).all())
    sure = ~torch.isnan(want)
    assert bool((got == want)[sure & torch.isinf(want)].all())
    sure &= ~torch.isinf(want)
    assert bool(((got - want).abs() <= want.abs() * 2.0 ** -8 + 4e-5)[sure].all())
    assert bool((c[M:] == 7).all()) and bool((c[:, -8:] == 7).all())


# The 64-wide tiles of the other kernel take their activations straight from the registers, the tanh form of GELU through LDS
@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (33, 40, 56), (130, 24, 200), (65, 248, 520)])
@pytest.mark.parametrize("tile", [39, 40, 41])
@pytest.mark.parametrize("kind,act,bias", [(BIAS_ACT, 0, True), (BIAS_ACT, 1, False), (ACT, 0, True), (ACT, 1, True), (DACT, 0, True), (DACT, 1, True),
                                           (DSWIGLU, 0, True), (ROPE, 0, True), (SWIGLU, 0, True), (SWIGLU, 0, False)])
def test_64_wide_tiles_give_what_128_square_ones_give(ctx, kind, act, bias, tile, M, N, K):
    if kind == ROPE and N < 144:
        N = 144
    gen = torch.Generator(device="cuda").manual_seed(82)
    g, c, c2, keep = _desc(kind, False, M, N, K, gen, bias, keep_c=bias or kind != SWIGLU)
    g.epi.act = (B.ACT_GELU_ERF, B.ACT_GELU_TANH)[act]
    _compare(ctx, g, c, c2, tile, M)
    if kind in (DACT, DSWIGLU) and tile == 39:      # dY W, whose second operand is K-slow: the only 64-wide shape of that form
        b = keep[1].t().contiguous()
        g.B, g.ldb, g.trans_b = b.data_ptr(), N, 1
        _compare(ctx, g, c, c2, tile, M)
    del keep
