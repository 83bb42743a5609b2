"""Which kernel a contraction runs on (csrc/gemm.hip), asked of the host functions that the launches themselves go by: what the rules take, and
every condition under which they must not.  Nothing is launched; addresses are made up."""
import ctypes as C

import pytest

from paper_2511_11641_amd import binding as B
from util import GemmDesc

STORE, BIAS_ACT, DACT, DSWIGLU, ACT, ROPE, SWIGLU = range(7)
FLOW, SHAPES = 12, 12
NONE, PAIR_BF16, PAIR_F32 = range(3)


@pytest.fixture(scope="module")
def lib():
    return B.load()


def _route(lib, g):
    return lib._Z17ecospa_gemm_routeRK8GemmDesc(C.byref(g))


def _pair(lib, w, x):
    return lib._Z22ecospa_gemm_pair_routeRK8GemmDescS1_PiS2_(C.byref(w), C.byref(x), C.byref(C.c_int()), C.byref(C.c_int()))


def _big(kind=STORE, tt=False, M=6144, N=6144, K=2048, **over):
    g = GemmDesc(B.BF16, M, N, K, 1 << 32, M if tt else K, int(tt), 2 << 32, N if tt else K, int(tt), 0, 1, None)
    g.epi.kind, g.epi.act, g.epi.c, g.epi.ldc = kind, B.ACT_GELU_ERF, 3 << 32, N
    for k, v in over.items():
        setattr(g.epi if hasattr(g.epi, k) else g, k, v)
    return g


@pytest.mark.parametrize("kind,tt", [(k, False) for k in range(7)] + [(STORE, True)])
def test_resident_workgroups_take_several_rounds_of_tiles(lib, kind, tt):
    assert _route(lib, _big(kind, tt)) == FLOW
    for over in (dict(K=2056), dict(K=960), dict(lda=1 << 23), dict(ldb=1 << 23), dict(ldc=1 << 23), dict(ldc2=1 << 23), dict(ldh=1 << 23),
                 dict(splits=2), dict(tile=35), dict(M=192 * 16, N=192 * 16), dict(trans_b=int(not tt))):
        assert 0 <= _route(lib, _big(kind, tt, **over)) < SHAPES, over
    if kind in (ACT, BIAS_ACT, DACT):
        assert _route(lib, _big(kind, act=B.ACT_GELU_TANH)) < SHAPES
    if tt:
        assert _route(lib, _big(tt=True, colsum=5 << 32)) < SHAPES
        assert _route(lib, _big(tt=True, bias=5 << 32)) < SHAPES


def _two(dt, T, d, n, w_tile=39, x_tile=38):
    """dW = dH^T X and dX = dH W over T tokens; every buffer apart from the others (tile codes: 64 x 128, 128 x 128)."""
    es, at = (2 if dt == B.BF16 else 4), iter(range(1 << 32, 99 << 32, 1 << 32))
    dh, x, wt, dw, dx = (next(at) for _ in range(5))
    w = GemmDesc(dt, n, d, T, dh, n, 1, x, d, 1, w_tile, 1, None)
    g = GemmDesc(dt, T, d, n, dh, n, 0, wt, n, 0, x_tile, 1, None)
    w.epi.c, w.epi.ldc, g.epi.c, g.epi.ldc = dw, d, dx, d
    ends = dict(dh=dh + T * n * es, x=x + T * d * es, wt=wt + d * n * es, dw=dw + n * d * es, dx=dx + T * d * es)
    return w, g, dict(dh=dh, x=x, wt=wt, dw=dw, dx=dx), ends


@pytest.mark.parametrize("dt,T,d,n,want", [(B.BF16, 1379, 264, 392, PAIR_BF16), (B.F32, 512, 256, 512, PAIR_F32)])
def test_pairs_need_buffers_apart_and_the_built_forms(lib, dt, T, d, n, want):
    w, x, p, end = _two(dt, T, d, n)
    assert _pair(lib, w, x) == want
    x.epi.c, w.epi.c = end["dw"], end["x"]                                   # side by side without a byte in common
    assert _pair(lib, w, x) == want

    def refused(change):
        w, x, p, end = _two(dt, T, d, n)
        change(w, x, p, end)
        assert _pair(lib, w, x) == NONE

    refused(lambda w, x, p, end: setattr(x.epi, "c", p["x"]))                # dX over X, which dW reads
    refused(lambda w, x, p, end: setattr(x.epi, "c", end["x"] - 16))         # ... over its last elements
    refused(lambda w, x, p, end: setattr(x.epi, "c", p["dh"]))
    refused(lambda w, x, p, end: setattr(x.epi, "c", end["dw"] - 16))
    refused(lambda w, x, p, end: setattr(w.epi, "c", end["wt"] - 16))        # dW over what dX reads
    refused(lambda w, x, p, end: setattr(w.epi, "c", end["dh"] - 16))
    refused(lambda w, x, p, end: setattr(w, "colsum", end["dx"] - 4))        # column sums over dX
    refused(lambda w, x, p, end: setattr(w, "colsum", p["wt"]))

    def side_input(w, x, p, end):                                            # dW over the saved pre-activations that dH reads
        x.epi.kind, x.epi.h, x.epi.ldh = DACT, end["dw"] - 16, d
    refused(side_input)
    refused(lambda w, x, p, end: setattr(x, "splits", 2))
    refused(lambda w, x, p, end: setattr(x, "trans_a", 1))
    refused(lambda w, x, p, end: setattr(w, "trans_b", 0))
    if dt == B.F32:
        w, x, *_ = _two(dt, 4096, 1024, 4096)                                # 64 x 64 tiles fill the chip
        assert _pair(lib, w, x) == NONE
        refused(lambda w, x, p, end: setattr(w, "splits", 2))
        return
    refused(lambda w, x, p, end: setattr(x, "trans_b", 1))
    refused(lambda w, x, p, end: setattr(x.epi, "kind", ACT))
    refused(lambda w, x, p, end: (setattr(w, "splits", 3), setattr(w, "partial", 50 << 32)))                  # its reduction not deferred
    w, x, p, end = _two(dt, T, d, n)
    w.splits, w.partial, w.defer_reduce = 3, 50 << 32, 1
    assert _pair(lib, w, x) == want
    x.epi.c = w.partial + 3 * n * d * 4 - 16                                 # dX over the partial sums
    assert _pair(lib, w, x) == NONE
    for over in ("lda", "ldb"):
        refused(lambda w, x, p, end: setattr(w, over, 1 << 23))
    refused(lambda w, x, p, end: setattr(x, "tile", 30))                     # 256 x 256 tiles: not built in a pair
    refused(lambda w, x, p, end: setattr(w, "tile", 30))
    w, x, *_ = _two(dt, 8192, 2048, 8192, 38, 38)                            # full rounds of tiles on both sides
    assert _pair(lib, w, x) == NONE
