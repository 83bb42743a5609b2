"""The contraction kernel of resident workgroups (csrc/gemm_flow.h) against the kernel of one tile per workgroup: every epilogue, tiles cut
off at both edges, two and three tiles per workgroup, the shortest K it takes and one that is no multiple of the ring's three slabs."""
import ctypes as C

import pytest
import torch

from paper_2511_11641_amd import binding as B
from util import GemmDesc

pytestmark = pytest.mark.gpu
STORE, BIAS_ACT, DACT, DSWIGLU, ACT, ROPE, SWIGLU = range(7)
FLOW = ("_Z19gemm_flow_launch_ntP10ecospa_ctxRK8GemmDesc", "_Z19gemm_flow_launch_ttP10ecospa_ctxRK8GemmDesc")
ROUTE, ROUTE_FLOW = "_Z17ecospa_gemm_routeRK8GemmDesc", 12
RING_192 = 35          # tile code: 192 x 192, one tile per workgroup


@pytest.fixture(scope="module")
def ctx():
    return B.Context("cuda:0")


def _rnd(gen, *shape):
    return torch.randn(*shape, device="cuda", generator=gen).bfloat16()


def _desc(kind, tt, M, N, K, gen, bias=True, keep_c=True):
    """A descriptor, its two outputs inside larger buffers of a marker value, and what has to stay alive."""
    a, b = _rnd(gen, K, M) if tt else _rnd(gen, M, K), _rnd(gen, K, N) if tt else _rnd(gen, N, K)
    b *= K ** -0.5
    wide = 2 * N if kind == DSWIGLU else N
    c, c2 = torch.full((M + 3, wide + 8), 7.0, device="cuda").bfloat16(), torch.full((M + 3, N + 8), 7.0, device="cuda").bfloat16()
    g = GemmDesc(B.BF16, M, N, K, a.data_ptr(), a.stride(0), int(tt), b.data_ptr(), b.stride(0), int(tt), 0, 1, None)
    g.epi.kind, g.epi.act, g.epi.c, g.epi.ldc = kind, B.ACT_GELU_ERF, c.data_ptr(), c.stride(0)
    keep = [a, b]
    if not keep_c:
        g.epi.c = None
    if bias and not tt and kind not in (DACT, DSWIGLU):
        keep.append(_rnd(gen, N))
        g.epi.bias = keep[-1].data_ptr()
    if kind in (BIAS_ACT, SWIGLU):
        g.epi.c2, g.epi.ldc2 = c2.data_ptr(), c2.stride(0)
    if kind in (DACT, DSWIGLU):
        keep.append(_rnd(gen, M, wide))
        g.epi.h, g.epi.ldh, g.epi.kp = keep[-1].data_ptr(), wide, N
    if kind == ROPE:      # 24-wide heads: four query heads on two key heads' tables, then a part that is not turned
        kp, hkv, L = 24, 2 * max(1, N // 240), 190
        hq = 2 * hkv
        cs, sn = (torch.rand(hkv, L, kp // 2, device="cuda", generator=gen) for _ in range(2))
        keep += [cs, sn]
        g.epi.rope_cos, g.epi.rope_sin, g.epi.rope_cols, g.epi.rope_kp, g.epi.rope_L, g.epi.rope_hq, g.epi.rope_qpk = (
            cs.data_ptr(), sn.data_ptr(), (hq + hkv) * kp, kp, L, hq, hq // hkv)
    return g, c, c2, keep


@pytest.mark.parametrize("M,N,K", [(3265, 3080, 1024), (3256, 6136, 1088), (8, 51400, 1152), (49160, 200, 1024)])
@pytest.mark.parametrize("kind,tt,bias,keep_c", [(STORE, False, True, True), (BIAS_ACT, False, True, True), (ACT, False, True, True), (DACT, False, True, True),
                                                 (DSWIGLU, False, True, True), (ROPE, False, True, True), (SWIGLU, False, True, True), (STORE, True, True, True),
                                                 # no bias; SWIGLU forward only: one of its two stores is left out
                                                 (STORE, False, False, True), (BIAS_ACT, False, False, True), (ACT, False, False, True),
                                                 (ROPE, False, False, True), (SWIGLU, False, False, False), (SWIGLU, False, True, False)])
def test_resident_workgroups_give_what_one_tile_per_workgroup_gives(ctx, kind, tt, bias, keep_c, M, N, K):
    if tt:
        M -= M % 8
    gen = torch.Generator(device="cuda").manual_seed(71)
    g, c, c2, keep = _desc(kind, tt, M, N, K, gen, bias, keep_c)
    assert getattr(ctx.lib, FLOW[tt])(ctx.h, C.byref(g)) == 0
    got, got2 = c.clone(), c2.clone()
    c.fill_(7.0)
    c2.fill_(7.0)
    g.tile = RING_192
    assert ctx.lib._Z11ecospa_gemmP10ecospa_ctxRK8GemmDesc(ctx.h, C.byref(g)) == B.OK
    for x, y in ((got, c), (got2, c2)):
        # products are added in the same order and the epilogues' arithmetic is written out: the same bits
        assert torch.equal(x, y)
        assert bool((x[M:] == 7).all()) and bool((x[:, -8:] == 7).all()), "written beyond the matrix"
    assert keep_c or bool((got == 7).all())


def test_the_rule_takes_it_and_refuses_what_it_is_not_built_for(ctx):
    gen = torch.Generator(device="cuda").manual_seed(72)
    g, c, c2, keep = _desc(BIAS_ACT, False, 6140, 3064, 1024, gen)
    run = lambda: ctx.lib._Z11ecospa_gemmP10ecospa_ctxRK8GemmDesc(ctx.h, C.byref(g))
    for act, flow in ((B.ACT_GELU_ERF, True), (B.ACT_GELU_TANH, False)):       # the tanh form stays with the other kernel
        g.epi.act, g.tile = act, 0
        assert (getattr(ctx.lib, ROUTE)(C.byref(g)) == ROUTE_FLOW) == flow
        assert run() == B.OK
        got = c2.clone()
        c2.fill_(7.0)
        g.tile = RING_192
        assert getattr(ctx.lib, ROUTE)(C.byref(g)) == 5      # 192 x 192 of the other kernel
        assert run() == B.OK
        assert torch.equal(got, c2)
