"""GPU parity of the attention forward pass of 128 queries per workgroup (many workgroups: every training batch) with the backward pass
behind it, against the fp64 oracle: every pair of head widths, with and without a mask, a ragged last tile behind full ones, shared
key/value heads.  Small batches take the forward kernel of 32-query tiles instead, so the batch is large here."""
import pytest

from test_gpu_attn import ctx, run_attn_case      # noqa: F401  (fixture and case runner)
from test_gpu_gqa import run_gqa_case

pytestmark = pytest.mark.gpu


def enough(Bsz, L, h, narrow):
    """Beyond the rule of the 32-query kernel: its workgroups, against all that are resident (twice that for long causal sequences)."""
    resident = 512 if narrow else 256
    return (L + 31) // 32 * h * Bsz > (2 * resident if L >= 512 else resident)


# both paddings of 32, 64 and 128 dims on either side; L = 200: a full query tile and 72 rows, three full key tiles and 8 keys
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh,k_qk,k_vo", [(64, 32, 32), (64, 19, 64), (64, 48, 20), (64, 64, 40), (128, 32, 128), (128, 64, 96),
                                          (128, 96, 32), (128, 128, 64), (128, 96, 96)])
def test_head_widths(ctx, dh, k_qk, k_vo, causal):      # noqa: F811
    Bsz = 42 if k_qk + k_vo <= 64 else 21
    assert enough(Bsz, 200, 2, k_qk + k_vo <= 64)
    run_attn_case(ctx, 73, Bsz, 200, 128, 2, dh, k_qk, k_vo, rope=False, causal=causal, wscale=3.0)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("L", [65, 128, 129, 197, 577])
def test_lengths(ctx, L, causal):                       # noqa: F811
    Bsz = 1 + (1024 if L >= 512 else 512) // ((L + 31) // 32 * 4)
    assert enough(Bsz, L, 4, True)
    run_attn_case(ctx, 74, Bsz, L, 128, 4, 64, 32, 32, rope=True, causal=causal, bias=False, wscale=3.0)


@pytest.mark.parametrize("h,hkv,k_qk,k_vo,rope,causal,L", [(8, 2, 32, 32, True, True, 381), (6, 3, 64, 64, False, False, 197), (8, 1, 24, 24, True, True, 130)])
def test_shared_key_heads(ctx, h, hkv, k_qk, k_vo, rope, causal, L):      # noqa: F811
    Bsz = 1 + 512 // ((L + 31) // 32 * h)
    assert enough(Bsz, L, h, k_qk + k_vo <= 64)
    run_gqa_case(ctx, h, hkv, 128, k_qk, k_vo, rope, causal, L, Bsz)
