"""Attention over rows so wide that the 64 rows of a key or query tile reach over 4 GB (the kernels carry 64-bit lane offsets from 2^25
elements per row on): 536000 heads of 16 | 64 dims, a full tile of 64 tokens and one of 8, against attention in fp32."""
import ctypes as C

import torch

import pytest

from paper_2511_11641_amd import binding as B

pytestmark = pytest.mark.gpu


def _off(got, want):
    """Relative error of every token's row (of the whole, by the row's own norm)."""
    return (got - want).norm(dim=-1) / want.norm(dim=-1)


def test_rows_of_34_million_elements():
    ctx = B.Context("cuda:0")
    L, d, h, kq, kv = 72, 8, 536000, 16, 64
    nqkv, nvo = h * (2 * kq + kv), h * kv
    assert 63 * 2 * nvo > 2 ** 32 and nqkv > nvo          # row 63 of every stream lies beyond 32 bits
    gen = torch.Generator(device="cuda").manual_seed(91)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen, dtype=torch.bfloat16)
    x, dy, wqkv, wo = rnd(L, d), rnd(L, d), rnd(nqkv, d) * 0.5, rnd(d, nvo)
    qkv, o, y, dx = (torch.empty(s, device="cuda", dtype=torch.bfloat16) for s in ((L, nqkv), (L, nvo), (L, d), (L, d)))
    lse = torch.empty(h, L, device="cuda")
    dwqkv, dwo = torch.empty_like(wqkv), torch.empty_like(wo)
    desc = B.BlockDesc(block=B.BLOCK_ATTN, dtype=B.BF16, B=1, L=L, d_model=d, h=h, kp_qk=kq, kp_vo=kv, causal=1, scale=0.25, w_qkv=wqkv.data_ptr(),
                       w_o=wo.data_ptr(), ld_wqkv=d, ld_wo=nvo, h_kv=h)
    sv = B.Saved(qkv=qkv.data_ptr(), o=o.data_ptr(), lse=lse.data_ptr())
    ctx.ecospa_coupled_fwd(desc, x, y, sv)
    ctx.ecospa_coupled_bwd(desc, x, dy, sv, dx, B.Grads(dw_qkv=dwqkv.data_ptr(), ld_dwqkv=d, dw_o=dwo.data_ptr(), ld_dwo=nvo))
    mask = torch.full((L, L), float("-inf"), device="cuda").triu(1)
    dx_want = torch.zeros(L, d, device="cuda")
    step = 8000
    for h0 in range(0, h, step):
        cols = [(h0 * kq, kq), (h * kq + h0 * kq, kq), (2 * h * kq + h0 * kv, kv)]                    # Q | K | V of these heads
        w = [wqkv[c:c + step * k].float() for c, k in cols]
        for wi, (c, k) in zip(w, cols):
            assert float(_off(qkv[:, c:c + step * k].float(), x.float() @ wi.t()).max()) < 2 ** -7
        q, k, v = (qkv[:, c:c + step * kk].reshape(L, step, kk).transpose(0, 1).float().contiguous() for c, kk in cols)
        p = torch.softmax(0.25 * torch.bmm(q, k.transpose(1, 2).contiguous()) + mask, dim=-1)
        rows = lambda t: t.transpose(0, 1).reshape(L, -1)
        # bf16 probabilities, outputs and gradients, fp32 sums: 4e-3 to 5e-3 of a row; a row of a tile read from elsewhere is 0.1 or more
        assert float(_off(o[:, h0 * kv:(h0 + step) * kv].float(), rows(torch.bmm(p, v))).max()) < 2e-2, f"O, heads from {h0}"
        wo_h = wo[:, h0 * kv:(h0 + step) * kv].float()
        do = (dy.float() @ wo_h).bfloat16().float().reshape(L, step, kv).transpose(0, 1).contiguous()
        dv = torch.bmm(p.transpose(1, 2).contiguous(), do)
        ds = p * (torch.bmm(do, v.transpose(1, 2).contiguous()) - (do * torch.bmm(p, v)).sum(-1, keepdim=True)) * 0.25
        for g, wi, (c, kk) in zip((torch.bmm(ds, k), torch.bmm(ds.transpose(1, 2).contiguous(), q), dv), w, cols):
            g = rows(g)
            dx_want += g @ wi
            got, want = dwqkv[c:c + step * kk].float(), g.t() @ x.float()
            assert float((got - want).norm() / want.norm()) < 2e-2, f"dW_qkv, columns from {c}"
    assert float(_off(dx.float(), dx_want).max()) < 2e-2
    want = dy.float().t() @ o.float()
    assert float((dwo.float() - want).norm() / want.norm()) < 2e-2
