"""GPU parity of the attention forward pass whose wavefronts share out the keys of a 32-query tile (few workgroups), at the
edges of its tiles: sequence lengths around multiples of 32 and 64, wavefronts without a key tile, every head width, and
both sides of the rule that chooses it - against the fp64 oracle; the backward pass reads the log-sum-exp it leaves."""
import pytest

from paper_2511_11641_amd import binding as B
from test_gpu_attn import run_attn_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return B.Context("cuda:0")


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("L", [64, 65, 96, 129, 255, 257, 321, 577])
def test_lengths(ctx, L, causal):
    run_attn_case(ctx, 70, 1, L, 128, 2, 64, 32, 32, rope=False, causal=causal)


@pytest.mark.parametrize("dh,k_qk,k_vo", [(64, 64, 64), (64, 32, 64), (64, 64, 24), (128, 96, 32), (128, 32, 128), (128, 64, 128),
                                          (128, 128, 64), (128, 128, 128)])
def test_head_widths(ctx, dh, k_qk, k_vo):
    run_attn_case(ctx, 71, 2, 333, 128, 2, dh, k_qk, k_vo, rope=True, causal=True, bias=False, wscale=3.0)


@pytest.mark.parametrize("Bsz,h", [(8, 8), (8, 9)])      # 512 workgroups, all resident; 576, the 128-query kernel
def test_both_sides_of_the_rule(ctx, Bsz, h):
    run_attn_case(ctx, 72, Bsz, 256, 64 * h, h, 64, 32, 32, rope=False, causal=True)
