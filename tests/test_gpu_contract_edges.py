"""GPU parity of the contraction kernels where they can go wrong: K that is no multiple of the 64-deep slab (the first slab takes
the remainder, zeroed in LDS beyond it), fewer slabs than the LDS ring holds, K splits with an uneven or empty last range, and
every tile shape with remainders of one 8-column group and one row - against a plain fp64 product of the same bf16 operands."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2511_11641_amd import binding as B
from paper_2511_11641_amd import synth
from test_gpu_attn import run_attn_case
from test_gpu_ffn import run_ffn_case
from test_gpu_contract_flow import ACT, BIAS_ACT, DACT, DSWIGLU, ROPE, STORE, SWIGLU, _desc
from test_gpu_contract_share import _compare
from util import GemmDesc, assert_close, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return B.Context("cuda:0")


def _case(seed, M, N, K, ta, tb):
    a = synth.round_to(synth.normal(seed, 300, (K, M) if ta else (M, K)), "bf16")
    b = synth.round_to(synth.normal(seed, 301, (K, N) if tb else (N, K)), "bf16")
    want = (a.T if ta else a).astype(np.float64) @ (b if tb else b.T).astype(np.float64)
    return dev(a, "bf16"), dev(b, "bf16"), a, want


# tile codes: 30 .. 38 name the nine shapes of at least 128 x 128; 0 is the library's choice
@pytest.mark.parametrize("tile", [0, 30, 31, 32, 33, 34, 35, 36, 37, 38])
@pytest.mark.parametrize("ta,tb,M,N,K", [
    (False, False, 257, 264, 8), (False, False, 129, 136, 72), (False, False, 61, 200, 456), (False, False, 385, 392, 200),
    (True, True, 264, 264, 1), (True, True, 136, 392, 63), (True, True, 264, 136, 191), (True, True, 392, 264, 257),
    (False, True, 257, 264, 72), (False, True, 70, 136, 200), (True, False, 264, 136, 136)])
def test_contract_k_remainders(ctx, ta, tb, M, N, K, tile):
    ga, gb, _, want = _case(61, M, N, K, ta, tb)
    got = ctx.ecospa_contract(ga, ta, gb, tb, tile=tile, splits=1)
    assert_close(got, want, "bf16", f"{M}x{N}x{K} tile {tile}")


@pytest.mark.parametrize("M,N,K,splits", [(64, 128, 4191, 0), (384, 768, 1379, 0), (264, 136, 191, 3), (136, 264, 70, 4),     # the last splits are empty
                                           (1000, 264, 1379, 5)])
def test_weight_gradient_with_column_sums_any_token_count(ctx, M, N, K, splits):
    ga, gb, a, want = _case(62, M, N, K, True, True)
    got, cs = ctx.ecospa_contract_colsum(ga, gb, splits=splits)
    assert_close(got, want, "bf16", "product")
    assert_close(cs, a.astype(np.float64).sum(axis=0), "f32", "column sums")
    again, cs2 = ctx.ecospa_contract_colsum(ga, gb, splits=splits)
    assert torch.equal(got, again) and torch.equal(cs, cs2)


# the shapes with a 64-wide side, which have no code at the entry point: 39 = 64x128, 40 = 128x64, 41 = 64x64 inside the library
@pytest.mark.parametrize("ta,tb,tile", [(0, 0, 39), (0, 0, 40), (0, 0, 41), (0, 1, 39), (1, 1, 39)])
@pytest.mark.parametrize("M,N,K,splits", [(64, 128, 8, 1), (72, 136, 72, 1), (8, 8, 200, 1), (200, 264, 456, 1), (136, 72, 1096, 3), (64, 64, 320, 1)])
def test_64_wide_shapes(ctx, ta, tb, tile, M, N, K, splits):
    if ta:
        K += 3 if K > 64 else -3          # K-slow operands take any K
    ga, gb, a, want = _case(69, M, N, K, ta, tb)
    out = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    parts = torch.empty((splits, M, N), dtype=torch.float32, device="cuda")
    g = GemmDesc(B.BF16, M, N, K, ga.data_ptr(), ga.stride(0), ta, gb.data_ptr(), gb.stride(0), tb, tile, splits, parts.data_ptr())
    g.epi.c, g.epi.ldc = out.data_ptr(), N
    rows = ctx.lib._Z23ecospa_gemm_colsum_rowsRK8GemmDesc(C.byref(g))
    assert rows == splits * -(-N // (64 if tile >= 40 else 128))
    cs = torch.full((rows, M), float("nan"), dtype=torch.float32, device="cuda")
    if ta and tb:
        g.colsum = cs.data_ptr()
    assert ctx.lib._Z11ecospa_gemmP10ecospa_ctxRK8GemmDesc(ctx.h, C.byref(g)) == B.OK
    assert_close(out, want, "bf16", f"{M}x{N}x{K}")
    if ta and tb:
        assert_close(cs.sum(dim=0), a.astype(np.float64).sum(axis=0), "f32", "column sums")


@pytest.mark.parametrize("M,N,K,split", [(8, 64, 2048, True), (61, 2048, 1024, False), (65, 72, 3000, True), (129, 5504, 520, False)])
def test_few_rows(ctx, M, N, K, split):
    assert (ctx.lib.ecospa_contract_workspace_bytes(B.BF16, M, N, K, 0) > 0) == split
    ga, gb, _, want = _case(63, M, N, K, False, False)
    assert_close(ctx.ecospa_contract(ga, False, gb, False, splits=1), want, "bf16", "unsplit")
    assert_close(ctx.ecospa_contract(ga, False, gb, False), want, "bf16", "library's choice")


def _shares(lib, M, N, K):
    f = lib._Z20ecospa_gemm_shares_kRK8GemmDesc
    g = GemmDesc(B.BF16, M, N, K, 1 << 32, K, 0, 2 << 32, K, 0, 0, 1, None)
    g.epi.ldc = N
    return f(C.byref(g)) & 1 == 1


# Layers of few tokens, whose contractions would be split along K: x W^T (and dY W from a transposed copy) shares K inside its workgroups where that
# is faster - all of a layer 2048 wide with 61 tokens - and goes in parts where K is long.  dY W from the matrix itself goes in parts either way.
def test_few_tokens_rotary_projection_in_parts(ctx):
    assert min(ctx.lib._Z24ecospa_gemm_token_splitsiii(61, n, k) for n, k in ((3072, 2048), (1024, 2048), (2048, 3072))) > 1
    assert _shares(ctx.lib, 61, 3072, 2048)
    run_attn_case(ctx, 75, 1, 61, 2048, 32, 64, 32, 32, rope=True, causal=True, bias=False, structure="pretrained", transposed=True)
    run_attn_case(ctx, 76, 1, 61, 2048, 32, 64, 32, 32, rope=False, causal=True, structure="pretrained")


@pytest.mark.parametrize("act,n,k", [("swiglu", 2800, 1400), ("gelu", 5461, 2730)])
def test_few_tokens_activations_in_parts(ctx, act, n, k):
    kp = (k + 63) // 64 * 64
    nh = 2 * kp if act == "swiglu" else kp
    assert min(ctx.lib._Z24ecospa_gemm_token_splitsiii(61, *nk) for nk in ((nh, 2048), (kp, 2048), (2048, nh))) > 1
    assert _shares(ctx.lib, 61, nh, 2048)
    run_ffn_case(ctx, 77, 1, 61, 2048, n, k, act, "bf16", structure="pretrained")
    run_ffn_case(ctx, 78, 1, 61, 2048, n, k, act, "bf16", structure="pretrained", transposed=True)


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("block", ["swiglu", "gelu", "attention"])
def test_layers_with_long_k_in_parts(ctx, block, transposed):
    """8192 wide, 33 tokens: Q|K|V with the rotation, W_1 with the activation and dY W_2 with its derivative, the epilogue behind the sum of the parts."""
    for n in {"swiglu": (128, 64), "gelu": (64,), "attention": (384,)}[block]:
        assert ctx.lib._Z24ecospa_gemm_token_splitsiii(33, n, 8192) > 1 and not _shares(ctx.lib, 33, n, 8192)
    if block == "attention":
        run_attn_case(ctx, 83, 1, 33, 8192, 4, 64, 32, 32, rope=True, causal=True, bias=False, structure="pretrained", transposed=transposed)
    else:
        run_ffn_case(ctx, 84, 1, 33, 8192, 160, 64, block, "bf16", structure="pretrained", transposed=transposed)


@pytest.mark.parametrize("splits", [2, 3, 8])
@pytest.mark.parametrize("M,N,K", [(1, 8, 520), (33, 40, 1032), (70, 144, 520)])
@pytest.mark.parametrize("kind,act,bias", [(STORE, 0, True), (BIAS_ACT, 0, True), (BIAS_ACT, 1, False), (ACT, 0, True), (ACT, 1, True), (DACT, 0, True),
                                           (DACT, 1, True), (DSWIGLU, 0, True), (ROPE, 0, True), (SWIGLU, 0, True), (SWIGLU, 0, False)])
def test_epilogues_behind_the_sum_of_parts(ctx, kind, act, bias, M, N, K, splits):
    """K in parts and the reduction that knows every epilogue, against the contraction in one part."""
    if kind == ROPE:
        M, N = max(M, 33), 144          # four query and two key heads of 24
    gen = torch.Generator(device="cuda").manual_seed(85)
    g, c, c2, keep = _desc(kind, False, M, N, K, gen, bias, keep_c=bias or kind != SWIGLU)
    g.epi.act = (B.ACT_GELU_ERF, B.ACT_GELU_TANH)[act]
    _compare(ctx, g, c, c2, 0, M, splits)
    del keep


# 32 x 32 tiles with K shared out over a workgroup, and 64 x 64 tiles once 512 of them exist; K below, at and beyond the groups of 32
# of a wavefront; rows and columns off every tile; fp32 sums of K products of N(0, 1) values: relative error about K^0.5 2^-24 < 3e-6
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, True), (True, False)])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (33, 31, 5), (64, 65, 127), (130, 70, 128), (97, 200, 1025), (1473, 1409, 70)])
def test_contract_f32_edges(ctx, ta, tb, M, N, K):
    a = synth.normal(64, 300, (K, M) if ta else (M, K))
    b = synth.normal(64, 301, (K, N) if tb else (N, K))
    want = (a.T if ta else a).astype(np.float64) @ (b if tb else b.T).astype(np.float64)
    assert_close(ctx.ecospa_contract(dev(a), ta, dev(b), tb, splits=1), want, "f32", f"{M}x{N}x{K}")
    if K > 64:
        assert_close(ctx.ecospa_contract(dev(a), ta, dev(b), tb, splits=3), want, "f32", f"{M}x{N}x{K} in three parts")


# no workspace, one that holds fewer splits than the library would take (8 for this shape), and enough
@pytest.mark.parametrize("parts", [0, 2, 8])
@pytest.mark.parametrize("ta,tb", [(False, False), (True, True)])
def test_own_split_is_limited_to_the_workspace(ta, tb, parts):
    M, N, K = 16, 24, 2048
    ga, gb, _, want = _case(65, M, N, K, ta, tb)
    ctx = B.Context("cuda:0")          # a context of its own: nothing attached yet
    assert ctx.lib.ecospa_contract_workspace_bytes(B.BF16, M, N, K, 0) == 8 * M * N * 4
    if parts:
        ctx.reserve(parts * M * N * 4)
    out = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")

    def call(splits):
        return ctx.lib.ecospa_contract(ctx.h, B.BF16, M, N, K, ga.data_ptr(), ga.stride(0), int(ta), gb.data_ptr(), gb.stride(0), int(tb),
                                       out.data_ptr(), N, None, 0, splits)

    assert call(0) == B.OK
    assert_close(out, want, "bf16", f"{parts} parts held")
    assert torch.equal(out, ctx.ecospa_contract(ga, ta, gb, tb, splits=max(parts, 1)))


# Rounding against fp64.  The error of n additions in one chain is about 1.8e-8 n^0.5 of a sum of N(0, 1) products; chains of 256 and
# the chain of their K / 256 (at most 128) sums: 1.8e-8 (256 + 128)^0.5 = 3.5e-7, whatever K is.
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, True)])
@pytest.mark.parametrize("M,N,K", [(1536, 1472, 8192), (768, 2704, 1500), (96, 80, 32768)])
def test_contract_f32_error_does_not_grow_with_k(ctx, ta, tb, M, N, K):
    gen = torch.Generator(device="cuda").manual_seed(68)
    a = torch.randn((K, M) if ta else (M, K), device="cuda", generator=gen)
    b = torch.randn((K, N) if tb else (N, K), device="cuda", generator=gen)
    want = (a.t() if ta else a).double() @ (b if tb else b.t()).double()
    got = ctx.ecospa_contract(a, ta, b, tb)
    assert float((got.double() - want).norm() / want.norm()) < 4.5e-7


# the workspace that the header asks for holds a row of sums per split; the contraction would leave one per split and tile column
@pytest.mark.parametrize("M,N,K,splits", [(136, 1048, 200, 1), (64, 392, 1379, 3), (72, 264, 4191, 0), (24, 8, 5, 1)])
def test_column_sums_in_the_least_workspace(M, N, K, splits):
    ga, gb, a, want = _case(66, M, N, K, True, True)
    ctx = B.Context("cuda:0")
    lib = ctx.lib
    parts = lib.ecospa_contract_workspace_bytes(B.BF16, M, N, K, splits)
    sp = max(1, parts // (M * N * 4))
    least = (sp * M * 4 + 255) // 256 * 256 + parts
    out, cs = torch.empty((M, N), dtype=torch.bfloat16, device="cuda"), torch.empty((M,), dtype=torch.float32, device="cuda")

    def call(tile=0, splits=splits):
        return lib.ecospa_contract_colsum(ctx.h, M, N, K, ga.data_ptr(), M, gb.data_ptr(), N, out.data_ptr(), N, cs.data_ptr(), tile, splits)

    assert call() == B.ERR_WORKSPACE
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")
    assert lib.ecospa_set_workspace(ctx.h, ws.data_ptr(), least) == B.OK
    assert call() == B.OK
    assert_close(out, want, "bf16", "product")
    assert_close(cs, a.astype(np.float64).sum(axis=0), "f32", "column sums")
    assert call(tile=14) == B.ERR_SHAPE and call(splits=sp + 1) == B.ERR_WORKSPACE


# rows more than 4 GB / 64 apart: a tile of 128 rows (K-contiguous) or 64 k (K-slow) spans more than 32 bits of offset
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, True), (True, False)])
def test_contract_leading_dimensions_beyond_32_bits(ctx, ta, tb):
    M, N, K = 104, 120, 112
    big = torch.empty((120, (1 << 26) + 8), dtype=torch.bfloat16, device="cuda")     # 16 GB; A, B and C are strips of its columns
    ga, gb, a, want = _case(67, M, N, K, ta, tb)
    sa, sb, sc = big[:ga.shape[0], 1000:1000 + ga.shape[1]], big[:gb.shape[0], 1 << 22:(1 << 22) + gb.shape[1]], big[:M, 1 << 25:(1 << 25) + N]
    sa.copy_(ga)
    sb.copy_(gb)
    for splits in (1, 2):
        sc.zero_()
        ctx.ecospa_contract(sa, ta, sb, tb, splits=splits, out=sc)
        assert_close(sc, want, "bf16", f"{splits} parts")
    if ta and tb:
        got, cs = ctx.ecospa_contract_colsum(sa, sb, splits=1)
        assert_close(got, want, "bf16", "product")
        assert_close(cs, a.astype(np.float64).sum(axis=0), "f32", "column sums")
