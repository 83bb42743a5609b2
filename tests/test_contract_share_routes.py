"""Which contractions share K out inside the workgroups (csrc/gemm.hip), asked of the host functions that the launches go by."""
import ctypes as C

import pytest

from paper_2511_11641_amd import binding as B
from test_contract_routes import ACT, FLOW, ROPE, SHAPES, STORE, SWIGLU, _big, _route, _two, lib      # noqa: F401

SHARE = FLOW + 1
SHARES_K = "_Z20ecospa_gemm_shares_kRK8GemmDesc"


@pytest.mark.parametrize("M,N,K", [(1, 768, 768), (17, 2048, 2752), (61, 3072, 2048), (61, 5504, 2048), (200, 2048, 2752), (512, 768, 768)])
@pytest.mark.parametrize("kind", [STORE, ACT, ROPE, SWIGLU])
def test_few_tokens_share_k(lib, kind, M, N, K):      # noqa: F811
    g = _big(kind, M=M, N=N, K=K)
    assert _route(lib, g) >= SHARE and getattr(lib, SHARES_K)(C.byref(g))
    for over in (dict(trans_b=1), dict(splits=2), dict(lda=1 << 23), dict(ldc=1 << 23), dict(tile=38)):
        assert 0 <= _route(lib, _big(kind, M=M, N=N, K=K, **over)) < SHAPES, over
    assert _route(lib, _big(STORE, tt=True, M=8 * ((M + 7) // 8), N=N, K=K)) < SHARE


@pytest.mark.parametrize("M,N,K", [(1024, 1024, 512), (1024, 2048, 1024), (1024, 1024, 2048), (4096, 5504, 2048), (32768, 64, 1024), (12017, 384, 768)])
def test_more_tokens_do_not(lib, M, N, K):      # noqa: F811
    assert _route(lib, _big(M=M, N=N, K=K)) < SHARE


def test_no_pair_where_k_would_be_split(lib):      # noqa: F811
    """dX beside dW over few tokens: the other kernel would split dX along K; it runs by itself with K shared out instead."""
    T, d, n = 61, 2048, 2752
    w, x, *_ = _two(B.BF16, T, d, n)
    x.tile = 0
    assert _route(lib, x) >= SHARE and lib._Z24ecospa_gemm_token_splitsiii(T, d, n) > 1
    assert lib._Z22ecospa_gemm_pair_routeRK8GemmDescS1_PiS2_(C.byref(w), C.byref(x), C.byref(C.c_int()), C.byref(C.c_int())) == 0


@pytest.mark.parametrize("M,N,K", [(17, 240, 2960), (61, 64, 2952), (61, 2480, 2736), (200, 1040, 3888), (33, 128, 2960), (61, 3072, 2048), (61, 512, 11008)])
def test_shared_or_in_parts_is_a_question_of_the_sizes(lib, M, N, K):      # noqa: F811
    """A block asks before it launches, where the epilogue may not be filled in yet: every kind has the answer of the plain store, and what is
    not split because it shares K does share it."""
    shares = getattr(lib, SHARES_K)
    want = shares(C.byref(_big(STORE, M=M, N=N, K=K))) & 1
    assert lib._Z24ecospa_gemm_token_splitsiii(M, N, K) > 1 and want == (K < 4096)
    for kind in range(7):
        g = _big(kind, M=M, N=N, K=K)
        assert shares(C.byref(g)) & 1 == want, kind
        assert not want or _route(lib, g) >= SHARE, kind
