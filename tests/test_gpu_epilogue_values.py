"""Epilogues of the contractions at the ends of the number range, on every route: one tile per workgroup, resident workgroups, the reduction
of a split K, fp32.  The operands are zeros and ones, so that the epilogue's input is known exactly."""
import ctypes as C

import pytest
import torch

from paper_2511_11641_amd import binding as B
from util import GemmDesc

pytestmark = pytest.mark.gpu
STORE, BIAS_ACT, DACT, DSWIGLU, ACT, ROPE, SWIGLU = range(7)
GEMM, FLOW_NT = "_Z11ecospa_gemmP10ecospa_ctxRK8GemmDesc", "_Z19gemm_flow_launch_ntP10ecospa_ctxRK8GemmDesc"
RING_192 = 35
SIZES = {"ring": (200, 200, 64), "split": (72, 136, 1024), "f32": (70, 136, 40), "flow": (3265, 3080, 1024)}


@pytest.fixture(scope="module")
def ctx():
    return B.Context("cuda:0")


def _launch(ctx, route, kind, N_out, set_epi):
    """c = A B^T with A and B zero (ones in the first k for the derivative kinds: acc = 1) through one route; set_epi fills the epilogue in."""
    M, N, K = SIZES[route]
    dt = torch.float32 if route == "f32" else torch.bfloat16
    a, b = torch.zeros(M, K, device="cuda", dtype=dt), torch.zeros(N, K, device="cuda", dtype=dt)
    if kind in (DACT, DSWIGLU):
        a[:, 0] = b[:, 0] = 1.0
    part = torch.empty(2, M, N, device="cuda") if route == "split" else None
    g = GemmDesc(B.F32 if route == "f32" else B.BF16, M, N, K, a.data_ptr(), K, 0, b.data_ptr(), K, 0, RING_192 if route == "ring" else 0,
                 2 if route == "split" else 1, part.data_ptr() if part is not None else None, 0)
    out = torch.full((M, N_out * N // 2), 7.0, device="cuda", dtype=dt)
    g.epi.kind, g.epi.act, g.epi.c, g.epi.ldc = kind, B.ACT_GELU_ERF, out.data_ptr(), out.stride(0)
    keep = set_epi(g, M, N, dt)
    assert getattr(ctx.lib, FLOW_NT if route == "flow" else GEMM)(ctx.h, C.byref(g)) == 0
    torch.cuda.synchronize()
    return out, keep


@pytest.mark.parametrize("route", list(SIZES))
@pytest.mark.parametrize("kind", [ACT, BIAS_ACT])
def test_gelu(ctx, route, kind):
    """x Phi(x): infinite for +inf, not a number for -inf (infinity times zero) and NaN."""
    def epi(g, M, N, dt):
        h = torch.tensor([float("-inf"), float("inf"), float("nan"), -3e38, 3e38, -20.0, 0.0, 1.5], device="cuda", dtype=dt).repeat(N // 8)
        c2 = torch.full((M, N), 7.0, device="cuda", dtype=dt)
        g.epi.bias, g.epi.c2, g.epi.ldc2 = h.data_ptr(), c2.data_ptr(), N
        return h, c2
    c, (h, c2) = _launch(ctx, route, kind, 2, epi)
    if kind == BIAS_ACT:
        assert bool(torch.equal(torch.nan_to_num(c, 9.0), torch.nan_to_num(h, 9.0).expand_as(c)))
        c = c2
    want = (h.double() * 0.5 * torch.special.erfc(-h.double() * 2 ** -0.5)).expand_as(c)
    assert bool((torch.isnan(c) == torch.isnan(want)).all())
    ok = ~torch.isnan(want)
    assert bool((torch.isinf(c) == torch.isinf(want))[ok].all())
    ok &= ~torch.isinf(want)
    assert float(((c - want).abs() - 2 ** -8 * want.abs())[ok].max()) <= 1e-30
