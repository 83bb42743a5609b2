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


@pytest.mark.parametrize("route", ["ring", "split", "flow"])
def test_gates_whose_sigmoid_is_below_the_normal_range(ctx, route):
    """exp(88) is a number, so gates down to -88.5 have a sigmoid (subnormal) and the products with it a value in the normal range."""
    gate = torch.tensor([-86.5, -87.5, -88.0, -88.5, -3.0, 90.0, 0.0, -100.0], device="cuda")
    sig = 1.0 / (1.0 + torch.exp(-gate.double()))
    sig[-1] = 0.0                                   # exp(100) overflows in fp32

    def fwd(g, M, N, dt):
        h = torch.stack((gate, torch.full_like(gate, 2.0)), 1).flatten().to(dt).repeat((N + 15) // 16)[:N].contiguous()
        act = torch.full((M, N // 2), 7.0, device="cuda", dtype=dt)
        g.epi.bias, g.epi.c2, g.epi.ldc2 = h.data_ptr(), act.data_ptr(), N // 2
        return h, act
    _, (_, act) = _launch(ctx, route, SWIGLU, 2, fwd)
    n = act.shape[1]
    want = (gate.double() * sig * 2.0).repeat((n + 7) // 8)[:n]
    # exp() of an argument of 88 is good to 88 * 2^-24, the bf16 rounding to 2^-9
    assert bool(((act.double() - want).abs() <= 2 ** -8 * want.abs()).all())

    def bwd(g, M, N, dt):
        h = torch.stack((gate, torch.full_like(gate, 2.0)), 1).flatten().to(dt).repeat((N + 7) // 8)[:2 * N].expand(M, 2 * N).contiguous()
        g.epi.h, g.epi.ldh, g.epi.kp = h.data_ptr(), 2 * N, N
        return h
    dh, _ = _launch(ctx, route, DSWIGLU, 4, bwd)
    n = dh.shape[1] // 2
    for half, w in ((0, 2.0 * sig * (1.0 + gate.double() * (1.0 - sig))), (1, gate.double() * sig)):
        want = w.repeat((n + 7) // 8)[:n]
        assert bool(((dh[:, half::2].double() - want).abs() <= 2 ** -8 * want.abs()).all())
