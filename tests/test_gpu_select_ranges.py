"""Top-k of groups whose scores share most of their bits, or none: where the radix passes of a large group start and end (csrc/select_dev.h)."""
import numpy as np
import pytest
import torch

from oracle import ecospa_oracle as O
from paper_2511_11641_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return B.Context("cuda:0")


def _neighbours(n, g, span):
    """Floats at most `span` steps apart."""
    return (np.float32(0.37).view(np.uint32) + g.integers(0, span + 1, n).astype(np.uint32)).view(np.float32)


SCORES = {
    "equal": lambda n, g: np.full(n, 0.25, np.float32),
    "one step apart": lambda n, g: _neighbours(n, g, 1),
    "255 steps apart": lambda n, g: _neighbours(n, g, 255),
    "256 steps apart": lambda n, g: _neighbours(n, g, 256),
    "2^20 steps apart": lambda n, g: _neighbours(n, g, 1 << 20),
    "spread norms": lambda n, g: np.exp(0.7 * g.standard_normal(n)).astype(np.float32) * np.float32(0.01),
    "every sign": lambda n, g: np.concatenate([[np.nan, np.inf, -np.inf, 0.0, -0.0, 1e-45, -1e-45], g.standard_normal(n - 7)]).astype(np.float32),
    "pairs": lambda n, g: np.repeat(g.standard_normal((n + 1) // 2), 2)[:n].astype(np.float32),
    "six in ten zero": lambda n, g: (np.exp(0.5 * g.standard_normal(n)) * (g.random(n) > 0.6)).astype(np.float32),
    "five values": lambda n, g: g.integers(0, 5, n).astype(np.float32),
    "two neighbours among others": lambda n, g: np.where(g.random(n) < 0.9, _neighbours(n, g, 1), 10.0 ** g.uniform(-30, 30, n) * g.choice((-1, 1), n)).astype(np.float32),
    "one above": lambda n, g: np.where(np.arange(n) == n // 2, 3e38, 1e-30).astype(np.float32),
}


@pytest.mark.parametrize("name", SCORES)
@pytest.mark.parametrize("n", [65, 1024, 1025, 8192, 8193, 32769])      # runs of 1, 2, 8, 9 units per thread and beyond the registers
def test_large_groups(ctx, n, name):
    g = np.random.default_rng(n)
    s = np.stack([g.permutation(SCORES[name](n, g)) for _ in range(2)])
    dev = torch.from_numpy(s).cuda()
    for k in (1, 2, n // 2, n - 1, n):
        got = ctx.ecospa_select_topk(dev, k).cpu().numpy()
        assert np.array_equal(got, O.select_topk(s, k)), f"{name}, {k} of {n}"
