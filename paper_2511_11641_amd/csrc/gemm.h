// Internal GEMM interface of the gfx950 library (not part of the C ABI).
//
//   C[m, n] = sum_k A(m, k) * B(n, k),   m < M, n < N, k < K
//   A(m, k) = A[m * lda + k]   (trans_a = 0, K contiguous)   or   A[k * lda + m]   (trans_a = 1)
//   B(n, k) = B[n * ldb + k]   (trans_b = 0, K contiguous)   or   B[k * ldb + n]   (trans_b = 1)
// so  X W^T  is (0, 0),  dY W  is (0, 1)  and  dY^T X  is (1, 1).
// Accumulation is fp32; the epilogue decides what is written.
#pragma once
#include "common.h"

enum {
  EPI_STORE = 0,     // c[m,n] = acc (+ bias[n])
  EPI_BIAS_ACT = 1,  // h = acc + bias[n]; c[m,n] = h; c2[m,n] = gelu(h)
  EPI_DACT = 2,      // c[m,n] = acc * gelu'(h[m,n])
  EPI_DSWIGLU = 3,   // unit n: g = h[m,2n], u = h[m,2n+1] (interleaved pairs); c[m,2n] = acc*u*dsilu(g); c[m,2n+1] = acc*silu(g)
  EPI_ACT = 4,       // c[m,n] = gelu(acc + bias[n]): forward only, the activation's input is not kept
  EPI_ROPE = 5,      // c[m,n] = acc + bias[n], with the adjacent column pairs (2i, 2i+1) of the first rope_cols columns
                     // turned by the angle of (row m % rope_L, pair) - the rotary form of the Q and K projections (bf16)
  EPI_SWIGLU = 6,    // columns come in (gate, up) pairs: h = acc (+ bias) is stored to c[m, n] (2 kp wide, when c is
                     // set) and silu(gate) * up to c2[m, n / 2] (kp wide) - the gated FFN's first contraction (bf16)
};

struct GemmEpi {
  int kind, act;
  void* c;
  long long ldc;
  const void* bias;
  void* c2;
  long long ldc2;
  const void* h;
  long long ldh;
  int kp;
  // EPI_ROPE: cos/sin tables float[rope_rows][rope_L][rope_kp / 2]; column n < rope_cols belongs to head n / rope_kp,
  // the query heads (the first rope_hq heads) share the table row of their key/value head: row head / rope_qpk for a
  // query head, head - rope_hq for a key head
  const float *rope_cos, *rope_sin;
  int rope_cols, rope_kp, rope_L, rope_hq, rope_qpk;
};

struct GemmDesc {
  int dtype;
  int M, N, K;
  const void* A;
  long long lda;
  int trans_a;
  const void* B;
  long long ldb;
  int trans_b;
  int tile;          // 0 = choose, otherwise a tile code of ecospa_contract, 39 .. 41 (64x128, 128x64, 64x64) or 50 .. 53 (gemm_share.h)
  int splits;        // > 1: split K, fp32 partials in `partial`, reduced in a fixed order
  float* partial;    // [splits][M][N] when splits > 1
  int defer_reduce;  // splits > 1: only write the partials; the caller runs ecospa_gemm_reduce later
  float* colsum;     // optional, contractions with a K-slow A operand (dY^T X; fp32: K unsplit): [ecospa_gemm_colsum_rows(d)][M] partial
                     // column sums of A, sum_k A(m, k) over disjoint parts of K - the bias gradient that belongs to the
                     // weight gradient, added up from the operand's fragments; the rows add up to the sums
  GemmEpi epi;
};

// Launch on ctx->stream.  bf16 and fp32 both run on MFMA tiles.
int ecospa_gemm(ecospa_ctx* ctx, const GemmDesc& d);
// Two contractions that do not depend on each other: w a weight gradient (dY^T X, bf16 or fp32; its reduction deferred where K is split), x
// over the same tokens.  One launch where that is built for the two and pays, otherwise w, then x (x_first: the other way round).
int ecospa_gemm_pair(ecospa_ctx* ctx, const GemmDesc& w, const GemmDesc& x, int x_first = 0);
// What the two above choose (host arithmetic only; they launch by it).  A bf16 contraction: the tile shape of the ring kernel, GEMM_ROUTE_FLOW
// for the kernel of resident workgroups, or GEMM_ROUTE_SHARE and a shape of the kernel that shares K out inside a workgroup.  A pair: one launch
// or two, and for one of bf16 the tile shapes.
int ecospa_gemm_route(const GemmDesc& d);
enum { GEMM_PAIR_NONE = 0, GEMM_PAIR_BF16 = 1, GEMM_PAIR_F32 = 2 };
int ecospa_gemm_pair_route(const GemmDesc& w, const GemmDesc& x, int* w_shape, int* x_shape);
// Rows (of M floats) of the partial column sums that the launch of d writes to d.colsum.
int ecospa_gemm_colsum_rows(const GemmDesc& d);
// Second half of a split-K contraction launched with defer_reduce: fixed-order sum of the partials,
// then the epilogue.  Same descriptor as the first half.
int ecospa_gemm_reduce(ecospa_ctx* ctx, const GemmDesc& d);
// How many K splits a (M, N, K) problem should use to fill the chip, and the bytes of partials.
int ecospa_gemm_splits(int dtype, int M, int N, int K);
// The same question for the contractions whose M is the token count (x W^T and dY W): with few tokens (inference
// at batch 1) their output has too few tiles for the chip; 1 for the training shapes.
int ecospa_gemm_token_splits(int M, int N, int K);
// Whether a contraction of few tokens is done sooner with K shared out inside the workgroups (gemm_share.h) than split over them.
bool ecospa_gemm_shares_k(const GemmDesc& d);

// The bf16 kernel (gemm_ring.h): launch of tile shape `shape` (index into the table in gemm.hip; not every shape is built for every
// form).  k_chunk: K range of a split, a multiple of 64.
#define GEMM_RING_NSHAPES 12
#define GEMM_ROUTE_FLOW GEMM_RING_NSHAPES
#define GEMM_ROUTE_SHARE (GEMM_RING_NSHAPES + 1)
#define GEMM_SHARE_NSHAPES 4
// Epilogue kinds that are built, as bit masks: x W^T carries all of them, dY W the activation derivatives, the forms with a K-slow A
// only the plain store.  (A split contraction leaves partial sums; the reduction behind it knows every kind.)
#define GEMM_EPIS_NT 0x7f
#define GEMM_EPIS_NN ((1 << EPI_STORE) | (1 << EPI_DACT) | (1 << EPI_DSWIGLU))
#define GEMM_EPIS_TX (1 << EPI_STORE)
static inline bool gemm_epi_built(int trans_a, int trans_b, int kind) {
  const int mask = trans_a ? GEMM_EPIS_TX : (trans_b ? GEMM_EPIS_NN : GEMM_EPIS_NT);
  return kind >= 0 && kind < 31 && ((mask >> kind) & 1);
}
// Leading dimensions from 2^23 on (256 rows of them are 4 GB): lane offsets of 64 bits, built for 128 x 128 tiles alone.
#define GEMM_RING_WIDE_SHAPE 8
static inline bool ring_wide(const GemmDesc& d) {
  const long long lim = 1ll << 23;
  return d.lda >= lim || d.ldb >= lim || d.epi.ldc >= lim || d.epi.ldc2 >= lim || d.epi.ldh >= lim;
}
// The kernel of resident workgroups (gemm_flow.h): x W^T with every epilogue but the tanh GELU, dY^T X without column sums; more tiles
// than compute units, whole slabs of K and enough of them to carry a tile's epilogue.
#define GEMM_FLOW_TILE 192
#define GEMM_FLOW_MIN_SLABS 16
static inline bool gemm_flow_takes(const GemmDesc& d) {
  const long long tiles = static_cast<long long>((d.M + GEMM_FLOW_TILE - 1) / GEMM_FLOW_TILE) * ((d.N + GEMM_FLOW_TILE - 1) / GEMM_FLOW_TILE);
  const bool act = d.epi.kind == EPI_BIAS_ACT || d.epi.kind == EPI_ACT || d.epi.kind == EPI_DACT;
  return d.splits <= 1 && !d.colsum && (d.trans_a != 0) == (d.trans_b != 0) && !(d.trans_a && d.epi.bias) && tiles > 256 && tiles < (1 << 24) &&
         d.K % 64 == 0 && d.K / 64 >= GEMM_FLOW_MIN_SLABS && !(act && d.epi.act != ECOSPA_ACT_GELU_ERF) && !ring_wide(d);
}
// The grid of a launch, worked out on the host: a workgroup finds its tile with multiplications.  What bounds a launch of few slabs is the
// time to its first load and what its XCD fetches from memory: six divisions one behind the other were 0.3 us of the 1.3 us to a workgroup's
// last first-round load, and bands of a fixed 16 tile rows had an XCD of 1024x1024x2048 on 64x64 tiles fetch 1152 operand rows where 768 do.
// The four contractions of a layer on 1024 tokens, 1024 wide, weights from memory: 41.5 -> 39.9 us with both and the bias asked for early.
// Workgroups are dealt round-robin to the 8 XCDs, each with an L2 of its own.  Every XCD gets a contiguous range of (K split, tile), so the
// tiles of one split, which read one K range of both operands, are on as few XCDs as there are.  Inside a split the tiles are ordered in
// bands of tile rows walked column by column, so that the tiles an XCD works on at a time form a block of C and share operand rows in
// its L2.
struct RingGrid {
  int tiles_n, k_chunk;
  int per, more;                  // workgroups per XCD; the first `more` XCDs have one more
  int tiles, group, band, last_band, last_rows;      // tiles of a split; rows and tiles of a band; where the last band starts, its rows
  unsigned tiles_inv, band_inv, group_inv, last_inv;
};
RingGrid gemm_ring_grid(int M, int N, int bm, int bn, int splits, int k_chunk);
hipError_t gemm_share_launch_nt(ecospa_ctx* ctx, const GemmDesc& d, int shape);
hipError_t gemm_flow_launch_nt(ecospa_ctx* ctx, const GemmDesc& d);
hipError_t gemm_flow_launch_tt(ecospa_ctx* ctx, const GemmDesc& d);
hipError_t gemm_ring_launch_nt(ecospa_ctx* ctx, const GemmDesc& d, int shape, int k_chunk);
hipError_t gemm_ring_launch_tt(ecospa_ctx* ctx, const GemmDesc& d, int shape, int k_chunk);
hipError_t gemm_ring_launch_mixed(ecospa_ctx* ctx, const GemmDesc& d, int shape, int k_chunk);
// Pairs (see ecospa_gemm_pair): by the weight gradient's tile rows; x on one of the shapes of GEMM_PAIR_X.
#define GEMM_PAIR_X ((1u << 4) | (1u << 5) | (1u << 7) | (1u << 8))
hipError_t gemm_pair_launch_64(ecospa_ctx* ctx, const GemmDesc& w, const GemmDesc& x, int x_shape, int w_k_chunk);
hipError_t gemm_pair_launch_128(ecospa_ctx* ctx, const GemmDesc& w, const GemmDesc& x, int x_shape, int w_k_chunk);
hipError_t gemm_pair_launch_192(ecospa_ctx* ctx, const GemmDesc& w, const GemmDesc& x, int x_shape, int w_k_chunk);
hipError_t gemm_pair_launch_256(ecospa_ctx* ctx, const GemmDesc& w, const GemmDesc& x, int x_shape, int w_k_chunk);

// The small jobs that follow the contractions of a backward pass, batched into ONE launch (each of
// them alone would be bound by the fixed cost of a launch): fixed-order reductions of split-K
// partials (a GemmDesc launched with defer_reduce) and bias gradients out[n] = sum_m X[m, n].
// A column sum is done by one workgroup per strip of columns over all rows - no second pass.
#define AUX_MAX_JOBS 4
#define AUX_OUT_F32 (-1)
struct AuxColsum {
  const void* X;
  long long ldx;
  int M, N, dtype;
  void* out;
  int out_dtype;     // 0: as X; ECOSPA_BF16 (fp32 partial sums reduced into a bf16 gradient); AUX_OUT_F32 (fp32 sums of a bf16 X)
};
struct AuxBatch {
  int n_reduce, n_colsum;
  GemmDesc reduce[AUX_MAX_JOBS];
  AuxColsum colsum[AUX_MAX_JOBS];
};
int ecospa_aux_launch(ecospa_ctx* ctx, const AuxBatch& b);

// Activation helpers shared by the epilogues and the elementwise kernels.
#ifdef __HIPCC__
// Tail of the standard normal distribution, Phi(-|x|), by the rational approximation 7.1.26 of Abramowitz & Stegun for erfc (absolute
// error about 3e-7 when evaluated in fp32: far below bf16 resolution, and a relative Frobenius error near 1e-7 on GELU outputs): one
// reciprocal, one exponential and a degree-5 Horner chain instead of the library erf, the factors 1/sqrt(2) and 1/2 folded into the
// constants.  `e` returns exp(-x^2 / 2), which the derivative needs as well.  GELU needs no comparison: x Phi(x) = max(x, 0) - |x| Phi(-|x|);
// the derivative's Phi(x) keeps one, or negative arguments would lose to cancellation.
// Vector instructions bound the activation epilogues: 15 and two transcendentals per element where the form with Phi itself took 20 (12017x768x384
// on 192x192 tiles, 13.4 us with a plain store: GELU 20.9 -> 19.4 us, with its argument kept 22.1 -> 21.2, the derivative 21.4 -> 20.9).
__device__ __forceinline__ float act_tail_t(float x) { return __builtin_amdgcn_rcpf(__builtin_fmaf(fabsf(x), 0.23164188f, 1.f)); }
__device__ __forceinline__ float act_gauss(float x) { return __builtin_amdgcn_exp2f(x * (x * -0.72134752f)); }
__device__ __forceinline__ float act_norm_tail(float x, float& e) {
  const float t = act_tail_t(x);
  float p = __builtin_fmaf(0.5307027145f, t, -0.7265760135f);
  p = __builtin_fmaf(p, t, 0.7107068705f);
  p = __builtin_fmaf(p, t, -0.142248368f);
  p = __builtin_fmaf(p, t, 0.127414796f);
  e = act_gauss(x);
  return p * t * e;
}
// (the bound keeps infinity times a tail of zero out of the positive side; x = -inf gives NaN, as x Phi(x) does)
__device__ __forceinline__ float act_gelu_of_tail(float x, float tail) { return __builtin_fmaf(-fabsf(fminf(x, 1e30f)), tail, fmaxf(x, 0.f)); }
__device__ __forceinline__ float act_gelu(float x, int act) {
  if (act == ECOSPA_ACT_GELU_TANH) {
    const float u = 0.7978845608028654f * (x + 0.044715f * x * x * x);
    return 0.5f * x * (1.f + tanhf(u));
  }
  float e;
  const float tail = act_norm_tail(x, e);
  return act_gelu_of_tail(x, tail);
}
__device__ __forceinline__ float act_gelu_grad(float x, int act) {
  if (act == ECOSPA_ACT_GELU_TANH) {
    const float u = 0.7978845608028654f * (x + 0.044715f * x * x * x);
    const float th = tanhf(u);
    return 0.5f * (1.f + th) + 0.5f * x * (1.f - th * th) * 0.7978845608028654f * (1.f + 0.134145f * x * x);
  }
  float e;
  const float tail = act_norm_tail(x, e);
  return __builtin_fmaf(x, 0.3989422804014327f * e, x < 0.f ? tail : 1.f - tail);
}
__device__ __forceinline__ float act_sigmoid(float x) { return 1.f / (1.f + __expf(-x)); }
// The same quotient in five instructions where the division takes ten: hardware reciprocal, one Newton step, special values.  1 + exp(-x)
// goes in at an eighth, so that no reciprocal falls below the normal range, where the hardware's is zero.  Equal to the division for every
// value of exp(-x) whose quotient is in the normal range (all tried on the card), within one step of the subnormal grid below it.  4096x5504x2048
// with SwiGLU: 89.6 us with this and with the division, 87.8 with the bare reciprocal (error 1.6 times as large); its derivative on
// 4096x2752x2048: 52.8 us with the division, 52.4 with this.
__device__ __forceinline__ float act_sigmoid_den(float e) { return __builtin_fmaf(e, 0.125f, 0.125f); }      // e = exp(-x)
__device__ __forceinline__ float act_sigmoid_step(float den, float r) { return __builtin_fmaf(__builtin_fmaf(-den, r, 1.f), r, r); }
__device__ __forceinline__ float act_sigmoid_end(float den, float r) { return __builtin_amdgcn_div_fixupf(r, den, 1.f) * 0.125f; }
__device__ __forceinline__ float act_sigmoid_rcp(float x) {
  const float den = act_sigmoid_den(__expf(-x));
  return act_sigmoid_end(den, act_sigmoid_step(den, __builtin_amdgcn_rcpf(den)));
}
#endif
