"""fp32 contractions whose workgroups are all resident at once run in a form of their own (csrc/gemm.hip: f32_few).  Its sums are those of the other
form in the same order: a launch of many workgroups and one of its first rows give the same bits, whatever the K range of a wavefront holds."""
import ctypes as C

import pytest
import torch

from paper_2511_11641_amd import binding as B
from util import GemmDesc

pytestmark = pytest.mark.gpu
STORE, BIAS_ACT, DACT, DSWIGLU, ACT = range(5)
GEMM, PAIR = "_Z11ecospa_gemmP10ecospa_ctxRK8GemmDesc", "_Z16ecospa_gemm_pairP10ecospa_ctxRK8GemmDescS3_i"
MANY, FEW, N = 990, 95, 830          # 806 and 78 tiles of 32 x 32 (three workgroups of the form reside on each of 256 compute units)


@pytest.fixture(scope="module")
def ctx():
    return B.Context("cuda:0")


def _desc(M, a, b, ta, tb, c, kind=STORE, h=None, c2=None, bias=None, colsum=None):
    K, n = (a.shape[0] if ta else a.shape[1]), (b.shape[1] if tb else b.shape[0])
    g = GemmDesc(B.F32, M, n, K, a.data_ptr(), a.stride(0), int(ta), b.data_ptr(), b.stride(0), int(tb), 0, 1, None)
    g.epi.kind, g.epi.act, g.epi.c, g.epi.ldc, g.epi.kp = kind, B.ACT_GELU_ERF, c.data_ptr(), c.stride(0), n
    if h is not None:
        g.epi.h, g.epi.ldh = h.data_ptr(), h.stride(0)
    if c2 is not None:
        g.epi.c2, g.epi.ldc2 = c2.data_ptr(), c2.stride(0)
    g.epi.bias = None if bias is None else bias.data_ptr()
    g.colsum = None if colsum is None else colsum.data_ptr()
    return g


@pytest.mark.parametrize("K", [1, 32, 127, 128, 160, 256, 300, 1025])
@pytest.mark.parametrize("ta,tb,kind", [(0, 0, STORE), (0, 0, BIAS_ACT), (0, 0, ACT), (0, 0, DACT), (0, 1, DACT), (0, 1, DSWIGLU), (0, 1, STORE), (1, 1, STORE), (1, 0, STORE)])
def test_many_workgroups_give_what_few_give(ctx, ta, tb, kind, K):
    gen = torch.Generator(device="cuda").manual_seed(K)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    a, b, bias = rnd(K, MANY) if ta else rnd(MANY, K), rnd(K, N) if tb else rnd(N, K), rnd(N)
    wide = 2 * N if kind == DSWIGLU else N
    h = rnd(MANY, wide)
    out = []
    for M in (MANY, FEW):
        c, c2, cs = torch.full((M + 1, wide + 4), 7.0, device="cuda"), torch.full((M + 1, N + 4), 7.0, device="cuda"), torch.full((M + 4,), 7.0, device="cuda")
        g = _desc(M, a, b, ta, tb, c, kind, h, c2, bias if kind not in (DACT, DSWIGLU) and not ta else None, cs if ta and tb else None)
        assert getattr(ctx.lib, GEMM)(ctx.h, C.byref(g)) == B.OK
        assert bool((c[M:] == 7).all()) and bool((c[:, wide:] == 7).all()) and bool((c2[M:] == 7).all()) and bool((cs[M:] == 7).all()), "written beyond"
        out.append((c[:FEW], c2[:FEW], cs[:FEW]))
    for x, y in zip(*out):
        assert torch.equal(x, y)
    if kind == STORE:
        want = (a.double().t() if ta else a.double())[:FEW] @ (b.double() if tb else b.double().t()) + (0 if ta else bias.double())
        assert float((out[0][0][:, :N].double() - want).norm() / want.norm()) < 3e-6      # fp32 sums: K^0.5 2^-24 at most


@pytest.mark.parametrize("T", [33, 300, 1025])
def test_pairs_of_many_workgroups_give_what_single_launches_give(ctx, T):
    """dW_2 | dH and dW_1 | dX, 512 workgroups and fewer (all resident in that form) and more, against the contractions one by one."""
    gen = torch.Generator(device="cuda").manual_seed(T)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    for d, n in ((64, 96), (200, 904)):
        dy, act, w2, hpre, x, w1 = rnd(T, d), rnd(T, n), rnd(d, n), rnd(T, n), rnd(T, d), rnd(n, d)
        new = lambda *s: torch.full(s, 7.0, device="cuda")
        res = []
        for pair in (True, False):
            dw2, dh, dw1, dx, s2, s1 = new(d, n), new(T, n), new(n, d), new(T, d), new(d), new(n)
            g = [_desc(d, dy, act, 1, 1, dw2, colsum=s2), _desc(T, dy, w2, 0, 1, dh, DACT, hpre)]
            k = [_desc(n, dh, x, 1, 1, dw1, colsum=s1), _desc(T, dh, w1, 0, 1, dx)]
            for w, y, first in ((*g, 1), (*k, 0)):
                if pair:
                    assert getattr(ctx.lib, PAIR)(ctx.h, C.byref(w), C.byref(y), first) == B.OK
                else:
                    assert getattr(ctx.lib, GEMM)(ctx.h, C.byref(w)) == B.OK and getattr(ctx.lib, GEMM)(ctx.h, C.byref(y)) == B.OK
            res.append((dw2, dh, dw1, dx, s2, s1))
        assert all(torch.equal(p, q) for p, q in zip(*res)), (d, n)
