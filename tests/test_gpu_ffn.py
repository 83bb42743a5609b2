"""GPU parity (through the C ABI) of the reduced FFN forward/backward against the fp64 oracle,
and of the whole chain score -> select -> compact -> fwd -> bwd on the fp32 single-pair workload."""
import numpy as np
import pytest
import torch

from oracle import ecospa_oracle as O
from paper_2511_11641_amd import binding as B
from paper_2511_11641_amd import synth
from paper_2511_11641_amd.layer import FfnBlock
from util import assert_close, dev, host, pad_cols, pad_rows, interleave_rows

pytestmark = pytest.mark.gpu

ACT = {"gelu": (B.ACT_GELU_ERF, O.ACT_GELU_ERF), "gelu_tanh": (B.ACT_GELU_TANH, O.ACT_GELU_TANH),
       "swiglu": (B.ACT_SWIGLU, O.ACT_SWIGLU)}


@pytest.fixture(scope="module")
def ctx():
    return B.Context("cuda:0")


def run_ffn_case(ctx, seed, Bsz, L, d, n, k, act, dtype, structure="scratch", bias=True, wscale=1.0, transposed=False):
    """Oracle scores/selects; both sides compact with the oracle's idx; compare everything."""
    gated = act == "swiglu"
    T = Bsz * L
    t = synth.ffn_layer(seed, T, d, n, gated=gated, dtype=dtype, structure=structure, bias=bias)
    if wscale != 1.0:
        for nm in ("w1", "w1b", "w2"):
            if nm in t:
                t[nm] = synth.round_to(t[nm] * np.float32(wscale), dtype)
    kind = O.PAIR_FFN_GATED if gated else O.PAIR_FFN
    v = O.coupled_score(kind, t["w1"], t["w2"], 1, n, w1b=t.get("w1b"))
    idx_np = O.select_topk(v.astype(np.float32), k)
    g = {nm: dev(a, dtype) for nm, a in t.items()}
    blk = FfnBlock(ctx, g["w1"], g.get("b1"), g["w2"], g.get("b2"), ACT[act][0], g.get("w1b"), transposed=transposed, bias_grads=True)
    blk.compact(torch.from_numpy(idx_np).cuda()).alloc(Bsz, L)
    kp = blk.kp
    y = blk.fwd(g["x"])
    dx = blk.bwd(g["x"], g["dy"])
    torch.cuda.synchronize()

    c = {nm: O.compact(t[nm], idx_np, 0, n) for nm in ("w1", "w1b", "b1") if nm in t}
    w2c = O.compact(t["w2"], idx_np, 1, n)
    yo, sv = O.ffn_fwd(t["x"], c["w1"], c.get("b1"), w2c, t.get("b2"), ACT[act][1], c.get("w1b"))
    go = O.ffn_bwd(t["x"], t["dy"], c["w1"], w2c, ACT[act][1], sv, c.get("w1b"))

    errs = {"y": assert_close(y, yo, dtype, "y"), "dx": assert_close(dx, go["dx"], dtype, "dx")}
    dw1 = pad_rows(go["dw1"], 1, k, kp)
    if gated:
        dw1 = interleave_rows(dw1, pad_rows(go["dw1b"], 1, k, kp))
    errs["dw1"] = assert_close(blk.dw1_c, dw1, dtype, "dw1")
    errs["dw2"] = assert_close(blk.dw2_c, pad_cols(go["dw2"], 1, k, kp), dtype, "dw2")
    db1 = pad_rows(go["db1"], 1, k, kp)
    if gated:
        # the up branch has no bias in the oracle; its column sums are sum_t dH_u
        db1 = interleave_rows(db1, pad_rows(_dhu_colsum(t, w2c, sv), 1, k, kp))
    errs["db1"] = assert_close(blk.db1_c, db1, dtype, "db1")
    errs["db2"] = assert_close(blk.db2, go["db2"], dtype, "db2")
    # padding slots hold exact zeros
    if kp > k:
        assert torch.all(blk.dw1_c[(2 * k if gated else k):] == 0) and torch.all(blk.dw2_c[:, k:] == 0)
    return errs


def _dhu_colsum(t, w2c, sv):
    da = np.asarray(t["dy"], np.float64) @ np.asarray(w2c, np.float64)
    h = sv["h"]
    return (da * h / (1.0 + np.exp(-h))).sum(axis=0)


@pytest.mark.parametrize("act", ["gelu", "gelu_tanh", "swiglu"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_ffn_small_ragged(ctx, act, dtype):
    # several tiles and ragged tails in every dimension: T=333, k=149 (kp=160)
    run_ffn_case(ctx, 21, 3, 111, 136, 301, 149, act, dtype, wscale=8.0)


@pytest.mark.parametrize("act,bias,transposed", [("gelu", True, False), ("swiglu", False, True)])
def test_ffn_long_token_axis_wide_weight_gradients(ctx, act, bias, transposed):
    """4096 tokens, 3072 kept units of 3200, d = 1024: weight gradients with enough 256x256 tiles that their
    contraction over the tokens fills the chip; the bias gradients are the column sums that it adds up on the way."""
    errs = run_ffn_case(ctx, 29, 4, 1024, 1024, 3200, 3072, act, "bf16", bias=bias, wscale=4.0, transposed=transposed)
    assert max(errs.values()) <= 2e-2


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
@pytest.mark.parametrize("dtype,T,d,n,k", [("bf16", 333, 136, 301, 149), ("bf16", 256, 2048, 4096, 2048), ("f32", 130, 72, 200, 99)])
def test_ffn_forward_only_keeps_nothing_and_agrees(ctx, act, dtype, T, d, n, k):
    """Forward without saved tensors (inference): the same output, bit for bit, as the training forward - the
    activation is computed from the same accumulators, only its input is not written."""
    gated = act == "swiglu"
    t = synth.ffn_layer(33, T, d, n, gated=gated, dtype=dtype)
    rng = np.random.default_rng(T)
    idx = torch.from_numpy(np.sort(rng.choice(n, k, replace=False)).astype(np.int32)[None, :]).cuda()
    g = {nm: dev(a, dtype) for nm, a in t.items()}
    blk = FfnBlock(ctx, g["w1"], g.get("b1"), g["w2"], g.get("b2"), ACT[act][0], g.get("w1b"), bias_grads=True)
    blk.compact(idx).alloc(1, T)
    y_train = blk.fwd(g["x"]).clone()
    blk.hpre.fill_(float("nan"))
    blk.act_buf.fill_(float("nan"))
    y_inf = blk.fwd(g["x"], save=False)
    assert torch.equal(y_inf, y_train)
    assert bool(torch.isnan(blk.hpre.float()).all()) and bool(torch.isnan(blk.act_buf.float()).all())   # untouched


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
def test_ffn_backward_with_optional_outputs(ctx, act):
    """Every gradient pointer is optional: the input gradient alone, the weight gradients without it, and bias
    gradients without their weight gradients (their own column-sum pass) equal what the full backward writes."""
    T, d, n, k = 520, 264, 400, 200
    t = synth.ffn_layer(34, T, d, n, gated=act == "swiglu", dtype="bf16")
    g = {nm: dev(a, "bf16") for nm, a in t.items()}
    idx = torch.from_numpy(np.sort(np.random.default_rng(5).choice(n, k, replace=False)).astype(np.int32)[None, :]).cuda()
    blk = FfnBlock(ctx, g["w1"], g.get("b1"), g["w2"], g.get("b2"), ACT[act][0], g.get("w1b"), bias_grads=True)
    blk.compact(idx).alloc(1, T)
    blk.fwd(g["x"])
    dx = blk.bwd(g["x"], g["dy"]).clone()
    full = {nm: getattr(blk, nm).clone() for nm in ("dw1_c", "dw2_c", "db1_c", "db2")}
    for nm in full:
        getattr(blk, nm).fill_(float("nan"))
    # input gradient only
    only_dx = torch.full_like(dx, float("nan"))
    ctx.ecospa_coupled_bwd(blk._desc, g["x"], g["dy"], blk.saved, only_dx, B.Grads())
    assert torch.equal(only_dx, dx)
    assert all(bool(torch.isnan(getattr(blk, nm).float()).all()) for nm in full)
    # everything but the input gradient
    ctx.ecospa_coupled_bwd(blk._desc, g["x"], g["dy"], blk.saved, None, blk.grads)
    for nm, want in full.items():
        assert torch.equal(getattr(blk, nm), want), nm
    # bias gradients without the weight gradients
    gr = B.Grads()
    gr.db_1, gr.db_2 = blk.db1_c.data_ptr(), blk.db2.data_ptr()
    blk.db1_c.fill_(float("nan")); blk.db2.fill_(float("nan"))
    ctx.ecospa_coupled_bwd(blk._desc, g["x"], g["dy"], blk.saved, None, gr)
    from util import TOL
    assert O.rel_fro(host(blk.db1_c), host(full["db1_c"])) <= TOL["bf16"] and O.rel_fro(host(blk.db2), host(full["db2"])) <= TOL["bf16"]


def test_ffn_weight_gradients_with_a_ragged_tile_row(ctx):
    """1100 kept units (padded to 1152 = 4.5 tiles of 256) at d = 2304 over 4096 tokens: the last tile row of the
    weight gradients is half empty, and its bias-gradient column sums must not count the columns beyond the edge twice."""
    errs = run_ffn_case(ctx, 32, 4, 1024, 2304, 1500, 1100, "gelu", "bf16", wscale=4.0)
    assert max(errs.values()) <= 2e-2


@pytest.mark.parametrize("act,bias", [("gelu", True), ("swiglu", True), ("swiglu", False)])
def test_ffn_weight_gradients_in_parts(ctx, act, bias):
    """1203 tokens, narrow matrices: both weight gradients are split along the tokens, their parts and the partial column sums of the
    bias gradients added up by the last launch."""
    nh = 800 if act == "swiglu" else 400
    assert min(ctx.lib._Z18ecospa_gemm_splitsiiii(B.BF16, m, n, 1203) for m, n in ((264, 400), (nh, 264))) > 1
    run_ffn_case(ctx, 35, 3, 401, 264, 700, 390, act, "bf16", bias=bias, wscale=4.0)


def test_ffn_wide_units_long_model_dimension(ctx):
    """4096 tokens, d = 2048, all 4096 units kept: x W_1^T and dY W_2 have a full round of 256x256 tiles with the bias +
    GELU epilogue (both outputs) and the GELU-derivative epilogue."""
    errs = run_ffn_case(ctx, 31, 4, 1024, 2048, 4096, 4096, "gelu", "bf16", wscale=3.0, transposed=True)
    assert max(errs.values()) <= 2e-2


@pytest.mark.parametrize("act,transposed", [("gelu", False), ("gelu", True), ("swiglu", True)])
def test_ffn_few_tokens_split_contractions(ctx, act, transposed):
    """256 tokens at d = 2048, 2048 kept units (inference at batch 1 and the like): the contractions have too few output tiles
    for the chip; the input gradient of the gated form (K = 4096) runs split along K, partial sums added in a fixed order."""
    run_ffn_case(ctx, 30, 1, 256, 2048, 4096, 2048, act, "bf16", wscale=4.0, transposed=transposed)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_ffn_keep_all_is_dense(ctx, dtype):
    run_ffn_case(ctx, 22, 2, 64, 64, 128, 128, "gelu", dtype, wscale=8.0)


def test_ffn_c1_fp32_whole_chain(ctx):
    """The fp32 single-pair workload: X[512x256], W_1[1024x256], W_2[256x1024], keep 512 of 1024.
    Here the GPU also scores and selects; indices must equal the oracle's on the GPU's scores and,
    for this seed, on the oracle's own scores too."""
    cfg = synth.CONFIGS["c1_ffn_f32"]
    T, d, n = cfg["T"], cfg["d"], cfg["n"]
    k = synth.keep_count(n, 1, 2)
    t = synth.ffn_layer(cfg["seed"], T, d, n, dtype="f32")
    g = {nm: dev(a) for nm, a in t.items()}
    blk = FfnBlock(ctx, g["w1"], g["b1"], g["w2"], g["b2"], B.ACT_GELU_ERF, bias_grads=True)
    sc = blk.score()
    want_sc = O.coupled_score(O.PAIR_FFN, t["w1"], t["w2"], 1, n)
    assert_close(sc, want_sc, "f32", "score")
    idx = ctx.ecospa_select_topk(sc, k)
    np.testing.assert_array_equal(idx.cpu().numpy(), O.select_topk(sc.cpu().numpy(), k))
    np.testing.assert_array_equal(idx.cpu().numpy(), O.select_topk(want_sc.astype(np.float32), k))
    errs = run_ffn_case(ctx, cfg["seed"], 1, T, d, n, k, "gelu", "f32")
    assert max(errs.values()) < 1e-5


@pytest.mark.parametrize("act,d,n,k,T", [("gelu", 1024, 4096, 2048, 1024), ("swiglu", 2048, 5461, 2730, 512)])
def test_ffn_model_shapes_bf16(ctx, act, d, n, k, T):
    """GPT-2-Medium and LLaMA-1B FFN widths at 50% keep (token count reduced to keep the oracle quick)."""
    run_ffn_case(ctx, 23, 2, T // 2, d, n, k, act, "bf16", structure="pretrained", bias=(act == "gelu"))


@pytest.mark.parametrize("act,d,n,k,T,dtype", [("gelu", 1024, 4096, 2048, 1024, "bf16"), ("swiglu", 2048, 5461, 2730, 512, "bf16"),
                                              ("gelu", 72, 200, 99, 130, "bf16"), ("gelu", 256, 1024, 512, 512, "f32")])
def test_ffn_backward_with_transposed_weight_copies(ctx, act, d, n, k, T, dtype):
    """The input-gradient contractions read transposed copies of the compact weights: same results to tolerance."""
    run_ffn_case(ctx, 17, 1, T, d, n, k, act, dtype, transposed=True)


def test_ffn_scattered_gradients_equal_masked_dense(ctx):
    """Scatter of the compact gradients = gradients of the dense layer with pruned rows/columns zeroed."""
    dtype, T, d, n, k = "f32", 96, 64, 80, 37
    t = synth.ffn_layer(24, T, d, n, dtype=dtype)
    v = O.coupled_score(O.PAIR_FFN, t["w1"], t["w2"], 1, n)
    idx_np = O.select_topk(v.astype(np.float32), k)
    idx = torch.from_numpy(idx_np).cuda()
    g = {nm: dev(a, dtype) for nm, a in t.items()}
    blk = FfnBlock(ctx, g["w1"], g["b1"], g["w2"], g["b2"], B.ACT_GELU_ERF, bias_grads=True).compact(idx).alloc(1, T)
    blk.fwd(g["x"])
    blk.bwd(g["x"], g["dy"])
    full_dw1 = ctx.ecospa_scatter(blk.dw1_c, idx, 0, 1, n, 1, blk.kp)
    full_dw2 = ctx.ecospa_scatter(blk.dw2_c, idx, 1, 1, n, 1, blk.kp)
    mask = np.zeros(n)
    mask[idx_np[0]] = 1
    _, sv = O.ffn_fwd(t["x"], t["w1"] * mask[:, None], t["b1"] * mask, t["w2"] * mask[None, :], t["b2"], O.ACT_GELU_ERF)
    gm = O.ffn_bwd(t["x"], t["dy"], t["w1"] * mask[:, None], t["w2"] * mask[None, :], O.ACT_GELU_ERF, sv)
    assert_close(full_dw1, gm["dw1"], dtype, "scattered dw1")
    assert_close(full_dw2, gm["dw2"] * mask[None, :], dtype, "scattered dw2")
    assert torch.all(full_dw1[torch.from_numpy(mask == 0).cuda()] == 0)


def test_ffn_is_deterministic(ctx):
    t = synth.ffn_layer(25, 512, 128, 256, dtype="bf16")
    g = {nm: dev(a, "bf16") for nm, a in t.items()}
    idx = torch.arange(0, 256, 2, dtype=torch.int32).view(1, -1).cuda()
    blk = FfnBlock(ctx, g["w1"], g["b1"], g["w2"], g["b2"], B.ACT_GELU_ERF, bias_grads=True).compact(idx).alloc(2, 256)
    outs = []
    for _ in range(2):
        blk.fwd(g["x"])
        blk.bwd(g["x"], g["dy"])
        outs.append([blk.y.clone(), blk.dx.clone(), blk.dw1_c.clone(), blk.dw2_c.clone(), blk.db1_c.clone()])
    for a, b in zip(*outs):
        assert torch.equal(a, b)
