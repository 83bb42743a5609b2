// Dense contractions of the reduced forward/backward pass: choice of kernel, tile shape and K split, the fp32 kernel, and the
// reductions of split contractions.
//
// bf16: the kernels of gemm_ring.h and, for several rounds of tiles, gemm_flow.h, for few tokens gemm_share.h (MFMA, direct global -> LDS loads).
// fp32: MFMA on fragments loaded straight from memory (the fp32 configuration is small and latency bound).
// Split-K writes fp32 partials that a second kernel adds in a fixed order (deterministic dW).
#include "gemm_epi.h"

// ---------------------------------------------------------------------------------------------
// fp32: v_mfma_f32_32x32x2_f32 on fragments that every lane loads straight from memory.  The fp32 problems are small: what bounds
// them is how many wavefronts there are and the latency of their loads, so nothing is staged through LDS.  A wavefront owns 32 x 32
// outputs; WK wavefronts of a workgroup share a tile's K and add up through LDS in a fixed order (WM = WN = 1), or the four form a
// 64 x 64 tile (WK = 1), whose operand rows are shared in the L1.  A chain of additions into one accumulator is at most F32_CHAIN
// products long, then its sum joins a second accumulator: the rounding error grows with the root of the chain (8192 products of
// N(0, 1) values in one chain: 1.6e-6 of the result, in chains of 256: 3.1e-7), for 16 additions per 128 matrix instructions.
// 512 x 512 x 256 (x W^T): vector-ALU kernel of 64 x 64 tiles through LDS 27 us, this one 6 us; 256 x 512 x 512 (dY^T X): 42 -> 8 us.
typedef float floatx16_f32 __attribute__((ext_vector_type(16)));
typedef float floatx4_f32 __attribute__((ext_vector_type(4), aligned(4)));

// 32 k of one operand row per lane pair: step j of lane half hh is k = 8 (j / 4) + 4 hh + j % 4 (both operands the same way)
template <bool KSLOW>
struct F32Frags {
  const float* p;      // this lane's row, k = 0
  long long ld;
  __device__ __forceinline__ void init(const void* mat, long long l, int row, int R) {
    ld = l;
    const int r = min(row, R - 1);
    p = static_cast<const float*>(mat) + (KSLOW ? r : r * l);
  }
  __device__ __forceinline__ void load(float (&v)[16], int k0, int hh) const {
    if constexpr (KSLOW) {
#pragma unroll
      for (int j = 0; j < 16; ++j) v[j] = p[(k0 + 8 * (j / 4) + 4 * hh + j % 4) * ld];
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const floatx4_f32 t = *reinterpret_cast<const floatx4_f32*>(p + k0 + 8 * q + 4 * hh);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[4 * q + i] = t[i];
      }
    }
  }
  __device__ __forceinline__ void load_tail(float (&v)[16], int k0, int k_end, int hh) const {     // zeros from k_end on
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int k = k0 + 8 * (j / 4) + 4 * hh + j % 4, kc = min(k, k_end - 1);
      const float t = KSLOW ? p[kc * ld] : p[kc];
      v[j] = k < k_end ? t : 0.f;
    }
  }
};

#define F32_CHAIN 256

// One output tile of K split z.  A K-slow A (dY^T X) also gives its column sums (GemmDesc::colsum, the bias gradient; K unsplit): the
// workgroups of the first tile column add the operand's values up as they pass, sixteen at a time in a tree, the sums of those with what their additions round away.
// FEW: for launches whose workgroups are all resident at once (f32_few), which last as long as one workgroup does.  The last pair of K groups then
// stands by itself, so that nothing is loaded twice; that takes 16 - 36 registers more, a workgroup less per compute unit.
template <int WM, int WN, int WK, bool TA, bool TB, bool FEW>
__device__ __forceinline__ void f32_tile(const GemmDesc& d, int tiles_n, int k_chunk, int block, int z) {
  static_assert(WM * WN * WK == 4 && (WK == 1 || WK == 4), "four wavefronts");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, hh = lane >> 5;
  const int wk = wave % WK, wmn = wave / WK, wm = wmn / WN, wn = wmn % WN;
  const int m0 = (block / tiles_n) * (32 * WM) + wm * 32, n0 = (block % tiles_n) * (32 * WN) + wn * 32;
  const int z0 = z * k_chunk, z1 = min(d.K, z0 + k_chunk);
  const int per = ((z1 - z0 + WK - 1) / WK + 31) / 32 * 32;       // K range of a wavefront: whole groups of 32
  const int k_begin = min(z0 + wk * per, z1), k_end = min(k_begin + per, z1);
  F32Frags<TA> fa;
  F32Frags<TB> fb;
  fa.init(d.A, d.lda, m0 + l32, d.M);
  fb.init(d.B, d.ldb, n0 + l32, d.N);
  floatx16_f32 acc, sum;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = sum[r] = 0.f;
  float a[2][16], b[2][16];
  const int nc = (k_end - k_begin) / 32;
  const bool sums = TA && TB && d.colsum && n0 == 0;
  float cs = 0.f, cs_lost = 0.f;
  auto products = [&](const float (&x)[16], const float (&y)[16]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 16; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[j], y[j], acc, 0, 0, 0);
    if (TA && TB && sums) {
      float t[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) t[j] = x[2 * j] + x[2 * j + 1];
      const float v = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7])), sum2 = cs + v, got = sum2 - cs;
      cs_lost += (cs - (sum2 - got)) + (v - got);       // what the addition rounded away
      cs = sum2;
    }
  };
  if (nc > 0) { fa.load(a[0], k_begin, hh); fb.load(b[0], k_begin, hh); }
  // The outputs that this lane writes: one column, NOUT rows.  What their epilogue reads besides the sums is asked for here; behind the
  // loop every output's saved pre-activation was a trip to memory of its own.  (Not for the 16 outputs of a lane of a 64 x 64 tile: 32 registers
  // more through the loop leave a SIMD two wavefronts where it has five; 1027x2448x192 with GELU' 32.5 us, 36.0 with them.)
  constexpr int NOUT = WK == 4 ? 4 : 16;
  constexpr bool AHEAD = WK == 4;
  auto row_out = [](int q) __attribute__((always_inline)) { return WK == 4 ? 8 * q : 8 * (q / 4) + q % 4; };
  const int m_out = m0 + (WK == 4 ? threadIdx.x >> 5 : 4 * hh), n_out = n0 + (WK == 4 ? threadIdx.x & 31 : l32);
  const bool derivative = (d.epi.kind == EPI_DACT || d.epi.kind == EPI_DSWIGLU) && d.splits <= 1, biased = d.splits <= 1 && d.epi.bias && !derivative;
  const int per_unit = d.epi.kind == EPI_DSWIGLU ? 2 : 1;
  float bias = 0.f, eh[NOUT], eu[NOUT];
#pragma unroll
  for (int q = 0; q < NOUT; ++q) eh[q] = eu[q] = 0.f;
  if (biased) bias = static_cast<const float*>(d.epi.bias)[min(n_out, d.N - 1)];
  auto side_column = [&]() __attribute__((always_inline)) { return static_cast<const float*>(d.epi.h) + static_cast<long long>(min(n_out, d.N - 1)) * per_unit; };
  if (AHEAD && derivative) {
    const float* const col = side_column();
#pragma unroll
    for (int q = 0; q < NOUT; ++q) {
      const float* const at = col + static_cast<long long>(min(m_out + row_out(q), d.M - 1)) * d.epi.ldh;
      eh[q] = at[0];
      eu[q] = at[per_unit - 1];
    }
  }
  // groups in pairs, no load behind a branch (the products of a pair would wait for it as well)
  int c = 0;
  auto chain_end = [&]() __attribute__((always_inline)) {
    if (c % (F32_CHAIN / 32) == 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) { sum[r] += acc[r]; acc[r] = 0.f; }
    }
  };
  if constexpr (FEW) {
    auto pair = [&](bool more) __attribute__((always_inline)) {
      fa.load(a[1], k_begin + (c + 1) * 32, hh);
      fb.load(b[1], k_begin + (c + 1) * 32, hh);
      products(a[0], b[0]);
      if (more) {
        fa.load(a[0], k_begin + (c + 2) * 32, hh);
        fb.load(b[0], k_begin + (c + 2) * 32, hh);
      }
      products(a[1], b[1]);
      c += 2;
      chain_end();
    };
    while (c + 2 < nc) pair(true);
    if (c + 2 == nc) pair(false);
  } else {
    while (c + 2 <= nc) {
      fa.load(a[1], k_begin + (c + 1) * 32, hh);
      fb.load(b[1], k_begin + (c + 1) * 32, hh);
      products(a[0], b[0]);
      const int kn = k_begin + min(c + 2, nc - 1) * 32;       // the last group again when there is no further one
      fa.load(a[0], kn, hh);
      fb.load(b[0], kn, hh);
      products(a[1], b[1]);
      c += 2;
      chain_end();
    }
  }
  if (c < nc) products(a[0], b[0]);
  if (k_begin + nc * 32 < k_end) {
    fa.load_tail(a[0], k_begin + nc * 32, k_end, hh);
    fb.load_tail(b[0], k_begin + nc * 32, k_end, hh);
    products(a[0], b[0]);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] += sum[r];
  float* part = d.splits > 1 ? d.partial + static_cast<long long>(z) * d.M * d.N : nullptr;
  if constexpr (TA && TB) {
    cs += fabsf(cs_lost) < INFINITY ? cs_lost : 0.f;      // (not a number behind an infinite sum, which stands as it is)
    cs += __shfl_xor(cs, 32, 64);      // the other half of the k
  }
  auto put = [&](int q, float v) __attribute__((always_inline)) {
    const int m = m_out + row_out(q);
    if (m < d.M && n_out < d.N) {
      if (!AHEAD && derivative) {
        const float* const at = side_column() + static_cast<long long>(m) * d.epi.ldh;
        eh[q] = at[0];
        eu[q] = at[per_unit - 1];
      }
      if (part) part[static_cast<long long>(m) * d.N + n_out] = v;
      else epi_put<float>(d.epi, m, n_out, biased ? v + bias : v, eh[q], eu[q]);
    }
  };
  // accumulator layout: column lane % 32, row 8 (r / 4) + 4 (lane / 32) + r % 4
  if constexpr (WK == 4) {
    __shared__ float red[4][32][33], red_cs[4][32];
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave][8 * (r / 4) + 4 * hh + r % 4][l32] = acc[r];
    if (TA && TB && hh == 0) red_cs[wave][l32] = cs;
    __syncthreads();
    if (TA && TB && sums && threadIdx.x < 32 && m0 + static_cast<int>(threadIdx.x) < d.M)
      d.colsum[m0 + threadIdx.x] = (red_cs[0][threadIdx.x] + red_cs[1][threadIdx.x]) + (red_cs[2][threadIdx.x] + red_cs[3][threadIdx.x]);
    const int n = threadIdx.x & 31;
#pragma unroll
    for (int q = 0; q < NOUT; ++q) {
      const int m = (threadIdx.x >> 5) + 8 * q;
      put(q, (red[0][m][n] + red[1][m][n]) + (red[2][m][n] + red[3][m][n]));
    }
  } else {
#pragma unroll
    for (int r = 0; r < NOUT; ++r) put(r, acc[r]);
    if (TA && TB && sums && hh == 0 && m0 + l32 < d.M) d.colsum[m0 + l32] = cs;
  }
}

template <int WM, int WN, int WK, bool TA, bool TB, bool FEW>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const GemmDesc d, int tiles_n, int k_chunk) {
  f32_tile<WM, WN, WK, TA, TB, FEW>(d, tiles_n, k_chunk, blockIdx.x, blockIdx.z);
}
// A weight gradient and a contraction over the tokens that do not depend on each other, in one launch: the first n_w workgroups take the
// tiles of the first.  Launches of this size last as long as one of their workgroups does, 6 - 8 us.
template <bool XTB, bool FEW>
__global__ __launch_bounds__(256) void gemm_f32_pair_kernel(const GemmDesc w, const GemmDesc x, int w_tiles_n, int n_w, int x_tiles_n) {
  const int block = blockIdx.x;
  if (block < n_w) f32_tile<1, 1, 4, true, true, FEW>(w, w_tiles_n, w.K, block, 0);
  else f32_tile<1, 1, 4, false, XTB, FEW>(x, x_tiles_n, x.K, block - n_w, 0);
}

// 64 x 64 tiles once they fill the compute units (half the operand traffic per product); below that K is what there is to share out
static bool f32_wide_tiles(const GemmDesc& d, int splits) {
  return static_cast<long long>((d.M + 63) / 64) * ((d.N + 63) / 64) * splits >= 512;
}

// Whether a compute unit takes all its workgroups of the launch at once in the FEW form as well: three by its registers, two of a pair.  512x512x256 with two
// outputs 6.0 us in the other form, 5.6 in this one; with more workgroups than are resident it is the other way round: dW_2 | dH of 512 tokens, 256 to 1024
// wide, 768 workgroups: 13.0 us, 15.8 in this one.
static bool f32_few(long long blocks, bool pair) { return blocks <= (pair ? 2 : 3) * 256; }

template <bool TA, bool TB>
static void launch_f32(ecospa_ctx* ctx, const GemmDesc& d, int splits) {
  const int k_chunk = (d.K + splits - 1) / splits;
  const int tm = (d.M + 63) / 64, tn = (d.N + 63) / 64, sm = (d.M + 31) / 32, sn = (d.N + 31) / 32;
  if (f32_wide_tiles(d, splits))
    hipLaunchKernelGGL((gemm_f32_kernel<2, 2, 1, TA, TB, false>), dim3(tm * tn, 1, splits), dim3(256), 0, ctx->stream, d, tn, k_chunk);
  else if (f32_few(static_cast<long long>(sm) * sn * splits, false))
    hipLaunchKernelGGL((gemm_f32_kernel<1, 1, 4, TA, TB, true>), dim3(sm * sn, 1, splits), dim3(256), 0, ctx->stream, d, sn, k_chunk);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<1, 1, 4, TA, TB, false>), dim3(sm * sn, 1, splits), dim3(256), 0, ctx->stream, d, sn, k_chunk);
}

// fixed-order sum of the K-split partials, then the epilogue
template <typename T>
__global__ __launch_bounds__(256) void gemm_splitk_reduce_kernel(const GemmDesc d) {
  const long long tot = static_cast<long long>(d.M) * d.N;
  const long long e = static_cast<long long>(blockIdx.x) * 256 + threadIdx.x;
  if (e >= tot) return;
  float s = 0.f;
  for (int z = 0; z < d.splits; ++z) s += d.partial[z * tot + e];
  epi_apply<T>(d.epi, static_cast<int>(e / d.N), static_cast<int>(e % d.N), s);
}
// bf16: 8 consecutive columns per thread (N is a multiple of 8)
__global__ __launch_bounds__(256) void gemm_splitk_reduce_vec8_kernel(const GemmDesc d) {
  const long long tot = static_cast<long long>(d.M) * d.N;
  const long long e = (static_cast<long long>(blockIdx.x) * 256 + threadIdx.x) * 8;
  if (e >= tot) return;
  float v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = 0.f;
  for (int z = 0; z < d.splits; ++z) {
    const float4 lo = *reinterpret_cast<const float4*>(d.partial + z * tot + e);
    const float4 hi = *reinterpret_cast<const float4*>(d.partial + z * tot + e + 4);
    v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w; v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
  }
  epi_apply_vec8(d.epi, static_cast<int>(e / d.N), static_cast<int>(e % d.N), v);
}

// ---------------------------------------------------------------------------------------------
// Kernel, tile shape and K split of a bf16 contraction.
//
// One workgroup per compute unit: a launch of the ring kernel takes rounds = ceil(tiles * splits / 256) of (slabs of 64 k) * slab + rest +
// epilogue, with slab and rest measured per shape on full rounds of 256 tiles (us; `rest`: first slabs from memory and the stores; 2 us
// more once per launch).  The K-slow forms read 8 bytes per LDS instruction instead of 16, which the narrow tiles feel most.  A split adds
// its partial sums: 3 us and their bytes at 4 TB/s; a split keeps at least 4 slabs.  The kernel of resident workgroups hides most of
// the rest and the epilogue of every tile but a workgroup's last.  The times are of operands that the L2s hold.  Those of the K-slow
// forms were taken when their LDS tiles still had bank conflicts; without, a slab takes 1.26 us on 256x256 tiles, 0.99 (192x256), 1.00, 0.72, 0.71, 0.79, 0.55,
// 0.56, 0.41 (128x128) and 0.31 (64x128), what lies beside the slabs up to 2 us less, and 0.80 with resident workgroups.  With operands from
// memory it takes 1.35, 1.19, 1.21, 0.74, 0.77, 0.78, 0.63, 0.64, 0.54 and 0.41.
//
// How good the choice is (the K-slow forms have not been tried like this): 680 contractions x W^T of random kinds and sizes (512 .. 32768 x 64 .. 52000
// x 256 .. 8300; activations just written, the rest from memory), every shape and the resident workgroups timed.  The sum over the choices is 1.0 - 1.4 % above the sum of the fastest, the worst
// single ones (fewer than 256 tiles, K beyond 3000) 1.4 times.  A slab of 256x256 is 1.28 us by least squares over the plain stores; with 1.30 or 1.33 in
// the table the sum is 0.1 - 0.7 % larger, with 0.79 - 0.83 for the resident workgroups' it is no smaller.  Outputs of more than 30000 columns
// cost those up to 3 us a round that the rule does not see (6144x24576x2048: 484 us, 440 on 256x256 tiles).
struct RingShape {
  int bm, bn;
  float slab_nt, slab_tt, rest;
};
static const RingShape RING_SHAPES[GEMM_RING_NSHAPES] = {
    {256, 256, 1.27f, 1.30f, 8.5f}, {192, 256, 1.05f, 1.03f, 6.5f}, {256, 192, 1.04f, 1.02f, 6.8f}, {128, 256, 0.73f, 0.74f, 5.2f},
    {256, 128, 0.71f, 0.73f, 5.4f}, {192, 192, 0.80f, 0.81f, 5.5f}, {128, 192, 0.54f, 0.57f, 4.3f}, {192, 128, 0.54f, 0.57f, 4.1f},
    {128, 128, 0.39f, 0.40f, 3.1f}, {64, 128, 0.26f, 0.29f, 2.2f},  {128, 64, 0.25f, 0.29f, 2.2f},  {64, 64, 0.165f, 0.20f, 1.7f}};
// Kernel of resident workgroups: per slab, per round beside it, and once.
static const float FLOW_SLAB_NT = 0.775f, FLOW_SLAB_TT = 0.79f, FLOW_ROUND = 2.3f, FLOW_REST = 6.0f;
// What an epilogue adds to a plain store, us per 1000 columns x rows of a tile (vector instructions and further outputs).
static float epi_us(int kind) {
  switch (kind) {
    case EPI_BIAS_ACT: case EPI_ACT: case EPI_DACT: return 0.23f;
    case EPI_SWIGLU: return 0.27f;
    case EPI_DSWIGLU: return 0.50f;
    case EPI_ROPE: return 0.15f;
    default: return 0.f;
  }
}
// Shapes that are built per form (bit i: shape i); see gemm_ring_*.hip.
static unsigned ring_shapes_built(int trans_a, int trans_b) {
  if (!trans_a && !trans_b) return 0xfffu;
  if (trans_a && trans_b) return 0x3ffu;        // at least 128 columns: the partial column sums have a row per tile column
  return trans_b ? 0x391u : 0x101u;
}
// Shape and split that finish soonest; splits > 0: that many, else 1 .. max_splits.  Returns the time (us).
static double ring_plan_search(int trans_a, int trans_b, int M, int N, int K, int kind, int splits, int max_splits, int* shape_out, int* splits_out) {
  const int slabs = (K + 63) / 64;
  const unsigned built = ring_shapes_built(trans_a, trans_b);
  double best = 0.0;
  int bs = -1, bq = 1;
  for (int q = 0; q < GEMM_RING_NSHAPES; ++q) {
    if (!((built >> q) & 1)) continue;
    const RingShape& r = RING_SHAPES[q];
    const long long tiles = static_cast<long long>((M + r.bm - 1) / r.bm) * ((N + r.bn - 1) / r.bn);
    const double slab = trans_a || trans_b ? r.slab_tt : r.slab_nt;
    const double epi = epi_us(kind) * r.bm * r.bn / 1000.0;
    for (int sp = splits > 0 ? splits : 1; sp <= (splits > 0 ? splits : max_splits); ++sp) {
      const int per = (slabs + sp - 1) / sp;                 // slabs of the first splits; the last one takes the rest
      if (splits <= 0 && sp > 1 && (per < 4 || per * (sp - 1) >= slabs)) break;
      const double mn = static_cast<double>(M) * N;
      const double red = sp > 1 ? 3.0 + (sp * mn * 4.0 + mn * 2.0) / 4.0e6 : 0.0;
      const double t = 2.0 + static_cast<double>((tiles * sp + 255) / 256) * (per * slab + r.rest + (sp > 1 ? 0.0 : epi)) + red;
      if (bs < 0 || t < best) { best = t; bs = q; bq = sp; }
    }
  }
  *shape_out = bs;
  *splits_out = bq;
  return best;
}
// The same from a table that each thread keeps of its latest questions (a function of the eight numbers alone).  A forward or backward call of a
// block asks thirty times - its workspace is laid out from the same answers - and 0.3 us each were half of the host time of such a call, which
// is what a few tokens wait for: attention and FFN block on 61 tokens, 2048 wide: enqueued in 23 us, with the table in 15.
static double ring_plan(int trans_a, int trans_b, int M, int N, int K, int kind, int splits, int max_splits, int* shape_out, int* splits_out) {
  struct Answer {
    int q[8];
    int shape, splits;
    double t;
  };
  static thread_local Answer table[128];      // all zeros: M = 0 is nobody's question
  const int q[8] = {trans_a, trans_b, M, N, K, kind, splits, max_splits};
  unsigned h = 0;
  for (int i = 0; i < 8; ++i) h = (h ^ static_cast<unsigned>(q[i])) * 0x9e3779b1u;
  Answer& a = table[h >> 25];
  if (memcmp(a.q, q, sizeof(q)) != 0) {
    a.t = ring_plan_search(trans_a, trans_b, M, N, K, kind, splits, max_splits, &a.shape, &a.splits);
    memcpy(a.q, q, sizeof(q));
  }
  *shape_out = a.shape;
  *splits_out = a.splits;
  return a.t;
}
static double flow_time(const GemmDesc& d) {
  const long long tiles = static_cast<long long>((d.M + GEMM_FLOW_TILE - 1) / GEMM_FLOW_TILE) * ((d.N + GEMM_FLOW_TILE - 1) / GEMM_FLOW_TILE);
  const double rounds = static_cast<double>(((tiles + 7) / 8 + 31) / 32);
  const double epi = epi_us(d.epi.kind) * GEMM_FLOW_TILE * GEMM_FLOW_TILE / 1000.0;
  return FLOW_REST + rounds * (d.K / 64 * (d.trans_a ? FLOW_SLAB_TT : FLOW_SLAB_NT) + FLOW_ROUND) + epi * (1.0 + 0.2 * (rounds - 1.0));
}

// Kernel that shares K out inside a workgroup: time of a round (us, weights from memory) and per unit of 64 k.  Against 1000 random contractions of 1 to
// 1100 rows, N and K 64 to 12000, every kind and shape: the time of a single round comes out 0.6 - 1.0 us short below K = 256, 0 - 0.4 short (spread
// 0.5) from 640 to 2048, 0.1 - 1.2 long (0.9 - 1.7) up to 4096 and 0.7 - 4 long beyond; a further round costs about as much as the first (512 tiles of 64x32
// at K = 512: 7.3 us, 64x64 of the ring kernel 4.9).
struct ShareShape {
  int bm, bn;
  float round, unit;
};
static const ShareShape SHARE_SHAPES[GEMM_SHARE_NSHAPES] = {{32, 16, 2.3f, 0.11f}, {32, 32, 2.2f, 0.155f}, {64, 16, 2.0f, 0.18f}, {64, 32, 2.3f, 0.215f}};
static bool gemm_share_takes(const GemmDesc& d) {
  return d.dtype == ECOSPA_BF16 && !d.trans_a && !d.trans_b && d.splits <= 1 && !d.colsum && !ring_wide(d);
}
static double share_plan(const GemmDesc& d, int kind, int* shape_out) {
  const int units = (d.K + 63) / 64;
  double best = 0.0;
  for (int q = 0; q < GEMM_SHARE_NSHAPES; ++q) {
    const ShareShape& r = SHARE_SHAPES[q];
    const long long tiles = static_cast<long long>((d.M + r.bm - 1) / r.bm) * ((d.N + r.bn - 1) / r.bn);
    const double t = static_cast<double>((tiles + 255) / 256) * (r.round + units * r.unit + epi_us(kind) * r.bm * r.bn / 1000.0);
    if (q == 0 || t < best) { best = t; *shape_out = q; }
  }
  return best;
}
// What the ring kernel takes beyond its table on 64-wide tiles, whose slabs the table has from L2.  Of the same contractions, weights from memory, 64x64
// tiles take nothing more below 4 slabs, 0.3 us at 4 - 8, 0.9 at 8 - 16, 2.1 at 16 - 24, 4.5 at 32 - 48 and 8.6 at 64 - 96, in parts 1.7 at 4 - 8 slabs, 2.5 at
// 8 - 16 and 4.1 at 16 - 24.  About half of that is counted: the kernel that shares K is then taken where it is faster and nowhere else - 830 of the 1000
// go to it, none of which the ring kernel, in parts or not, does sooner, weights in the caches or not; 40 with K from 2900 to 6700 stay in parts that would take 0.7 -
// 0.9 of the time.  The sum over the choices is 2 % above the sum of the fastest, 35 % without the kernel.
static double ring_cold(int shape, int slabs) { return shape >= 9 ? 0.065 * slabs - 0.6 : 0.0; }

int ecospa_gemm_splits(int dtype, int M, int N, int K) {
  if (dtype != ECOSPA_BF16) return 1;      // the fp32 kernel shares K out inside a workgroup
  int shape, sp;
  ring_plan(1, 1, M, N, K, EPI_STORE, 0, 8, &shape, &sp);
  return sp;
}

int ecospa_gemm_token_splits(int M, int N, int K) {
  int shape, sp;
  ring_plan(0, 0, M, N, K, EPI_STORE, 0, 8, &shape, &sp);
  return sp;
}

// A question of the sizes alone, like that for the split: both sides have the epilogue behind their sums, spread over the chip.  (The table prices
// none behind a split.  With its price on this side only, about one contraction in sixty with another epilogue than the plain store was split, K 2500 to
// 4800: 80 of those of every kind take 1.04 - 1.59 times as long in parts, 1.32 in the geometric mean; 61x2480x2736 with GELU' 13.1 us, shared 10.8.)
bool ecospa_gemm_shares_k(const GemmDesc& d) {
  if (!gemm_share_takes(d)) return false;
  int shape, sp, share;
  const double t = ring_plan(0, 0, d.M, d.N, d.K, EPI_STORE, 0, 8, &shape, &sp);
  return share_plan(d, EPI_STORE, &share) < t + ring_cold(shape, ((d.K + 63) / 64 + sp - 1) / sp);
}

// Rows of a band of tiles (gemm.h).  A launch of one round (256 tiles or fewer): an XCD's tiles of it are all under way together, and the height
// taken has the fewest operand rows per tile, the lower last band weighed in; heights up to 16, equal bands, the lowest of equals.  Without the
// last band 548x3200x3504 on 128x64 tiles, five tile rows, ran in bands of three and two: 32.9 us, 29.7 in one band; some 600 random launches of one
// round take 0.6 % less than in bands of 4, 8 or 16 (by tile height).  Those stay for several rounds, where the count says nothing of what the
// L2s keep from one to the next: 3632x5648x584 on 192x256 tiles 41.9 us in bands of 4, 46.1 of 7; 16345x1560x1496 on 256x256 88.2 of 4, 105 of 8.
static int ring_band_rows(int tiles_m, int bm, int bn, int blocks) {
  if (blocks > 256) {
    const int rows = bm >= 192 ? 4 : (bm >= 128 ? 8 : 16);
    return rows < tiles_m ? rows : tiles_m;
  }
  const int at_once = blocks < 8 ? 1 : blocks >> 3;
  const auto fetched = [&](int rows) { return rows * (rows * bm + (at_once + rows - 1) / rows * bn); };      // by the tile rows of a band
  int best = 1, fewest = 0;
  for (int rows = 1; rows <= 16 && rows <= tiles_m; ++rows) {
    const int bands = (tiles_m + rows - 1) / rows;
    if ((tiles_m + bands - 1) / bands != rows) continue;
    const int sum = (bands - 1) * fetched(rows) + fetched(tiles_m - (bands - 1) * rows);
    if (fewest == 0 || sum < fewest) { fewest = sum; best = rows; }
  }
  return best;
}
static unsigned ring_inverse(unsigned d) { return d <= 1 ? ~0u : static_cast<unsigned>((1ull << 32) / d); }
RingGrid gemm_ring_grid(int M, int N, int bm, int bn, int splits, int k_chunk) {
  RingGrid g;
  const int tiles_m = (M + bm - 1) / bm;
  g.tiles_n = (N + bn - 1) / bn;
  g.k_chunk = k_chunk;
  g.tiles = tiles_m * g.tiles_n;
  const int nb = g.tiles * splits;
  g.per = nb >> 3;
  g.more = nb & 7;
  g.group = ring_band_rows(tiles_m, bm, bn, nb);
  g.band = g.group * g.tiles_n;
  g.last_band = (tiles_m - 1) / g.group;
  g.last_rows = tiles_m - g.last_band * g.group;
  g.tiles_inv = ring_inverse(g.tiles);
  g.band_inv = ring_inverse(g.band);
  g.group_inv = ring_inverse(g.group);
  g.last_inv = ring_inverse(g.last_rows);
  return g;
}

// Workgroup tile that a tile code names, or 0: those of the contraction entry point, and 39 .. 41 for the 64-wide shapes.
static void ring_forced_tile(int tile, int* bm, int* bn) {
  static const int cfg[11][2] = {{256, 256}, {256, 256}, {256, 128}, {128, 256}, {128, 128}, {256, 256}, {128, 128}, {256, 256}, {256, 256}, {256, 128}, {256, 192}};
  static const int wg[12][2] = {{256, 256}, {192, 256}, {256, 192}, {128, 256}, {256, 128}, {192, 192},
                                {128, 192}, {192, 128}, {128, 128}, {64, 128}, {128, 64}, {64, 64}};
  *bm = *bn = 0;
  if (tile >= 1 && tile <= 4) { *bm = *bn = tile & 1 ? 128 : 256; }
  else if (tile >= 10 && tile <= 19) { *bm = cfg[tile - 10][0]; *bn = cfg[tile - 10][1]; }
  else if (tile == 20) { *bm = *bn = 256; }
  else if (tile == 21) { *bm = cfg[10][0]; *bn = cfg[10][1]; }
  else if (tile >= 30 && tile < 42) { *bm = wg[tile - 30][0]; *bn = wg[tile - 30][1]; }
}

// Shape of the ring kernel for d and the time it is expected to take (us; 0: not a choice of time).
static int ring_shape(const GemmDesc& d, int splits, double* t) {
  int shape, sp, bm, bn;
  *t = 0.0;
  if (ring_wide(d)) return GEMM_RING_WIDE_SHAPE;
  ring_forced_tile(d.tile, &bm, &bn);
  const unsigned built = ring_shapes_built(d.trans_a, d.trans_b);
  for (int q = 0; q < GEMM_RING_NSHAPES && bm; ++q)
    if (((built >> q) & 1) && RING_SHAPES[q].bm == bm && RING_SHAPES[q].bn == bn) return q;
  *t = ring_plan(d.trans_a, d.trans_b, d.M, d.N, d.K, d.epi.kind, splits, splits, &shape, &sp);
  return shape;
}

// Rows of the partial column-sum matrix (GemmDesc::colsum) that the launch of d writes, M floats each: one per K split and
// tile column.  The caller sizes the buffer with it and adds the rows up in order.
int ecospa_gemm_colsum_rows(const GemmDesc& d) {
  const int splits = d.splits > 1 ? d.splits : 1;
  if (d.dtype != ECOSPA_BF16) return splits;
  double t;
  const int bn = RING_SHAPES[ring_shape(d, splits, &t)].bn;
  return splits * ((d.N + bn - 1) / bn);
}

// What a descriptor has to satisfy before anything is launched.
static int gemm_check(const GemmDesc& d) {
  if (d.M < 1 || d.N < 1 || d.K < 1) return ECOSPA_ERR_SHAPE;
  if (!d.A || !d.B || (!d.epi.c && d.epi.kind != EPI_SWIGLU)) return ECOSPA_ERR_NULL;      // the gated epilogue may skip its first output
  if (d.splits > 1 && !d.partial) return ECOSPA_ERR_WORKSPACE;
  if (d.colsum && !(d.trans_a && d.trans_b && (d.dtype == ECOSPA_BF16 || d.splits <= 1))) return ECOSPA_ERR_SHAPE;      // column sums of A: the dY^T X form
  if (d.dtype == ECOSPA_F32) return d.epi.kind < EPI_STORE || d.epi.kind > EPI_ACT ? ECOSPA_ERR_DTYPE : ECOSPA_OK;      // the rotary and gated forms are bf16 only
  if (d.dtype != ECOSPA_BF16) return ECOSPA_ERR_DTYPE;
  // 16-byte vector loads along the contiguous axis of each operand
  const int ca = d.trans_a ? d.M : d.K, cb = d.trans_b ? d.N : d.K;
  if (ca % 8 || cb % 8 || d.lda % 8 || d.ldb % 8) return ECOSPA_ERR_ALIGN;
  if (!aligned16(d.A) || !aligned16(d.B)) return ECOSPA_ERR_ALIGN;
  // the epilogue moves 8 columns at a time
  if (d.N % 8 || d.epi.ldc % 8 || !aligned16(d.epi.c)) return ECOSPA_ERR_ALIGN;
  if (d.epi.kind == EPI_SWIGLU && (!d.epi.c2 || d.epi.ldc2 % 4 || (reinterpret_cast<uintptr_t>(d.epi.c2) & 7u))) return ECOSPA_ERR_ALIGN;
  if (d.epi.kind == EPI_ROPE && (!d.epi.rope_cos || !d.epi.rope_sin || !aligned16(d.epi.rope_cos) || !aligned16(d.epi.rope_sin) ||
                                 d.epi.rope_kp % 8 || d.epi.rope_cols % 8 || d.epi.rope_L < 1 || d.epi.rope_qpk < 1)) return ECOSPA_ERR_ALIGN;
  if (d.epi.bias && !aligned16(d.epi.bias)) return ECOSPA_ERR_ALIGN;
  if (d.epi.kind == EPI_BIAS_ACT && (!d.epi.c2 || d.epi.ldc2 % 8 || !aligned16(d.epi.c2))) return ECOSPA_ERR_ALIGN;
  if ((d.epi.kind == EPI_DACT || d.epi.kind == EPI_DSWIGLU) && (!d.epi.h || d.epi.ldh % 8 || !aligned16(d.epi.h)))
    return ECOSPA_ERR_ALIGN;
  if (d.epi.kind == EPI_DSWIGLU && d.epi.kp % 8) return ECOSPA_ERR_ALIGN;
  if (d.splits > 1 && !aligned16(d.partial)) return ECOSPA_ERR_ALIGN;
  if (!gemm_epi_built(d.splits > 1 ? 0 : d.trans_a, d.splits > 1 ? 0 : d.trans_b, d.epi.kind)) return ECOSPA_ERR_DTYPE;
  return ECOSPA_OK;
}

// K range of a split: whole 64-deep slabs, the last split takes what is left
static int ring_chunk(const GemmDesc& d, int splits) { return ((d.K + 63) / 64 + splits - 1) / splits * 64; }

// Timing window of ecospa_profile_gemm: events around a launch and the operations it does.
static bool prof_begin(ecospa_ctx* ctx) {
  const bool on = ctx->prof_on && ctx->prof_n < ctx->prof_cap;
  if (on) (void)hipEventRecord(ctx->prof_ev[2 * ctx->prof_n], ctx->stream);
  return on;
}
static void prof_end(ecospa_ctx* ctx, double flop) {
  (void)hipEventRecord(ctx->prof_ev[2 * ctx->prof_n + 1], ctx->stream);
  ctx->prof_flop[ctx->prof_n++] = flop;
}

// Ring kernel or resident workgroups.
static int tiled_route(const GemmDesc& d, double* t) {
  const int shape = ring_shape(d, d.splits > 1 ? d.splits : 1, t);
  return gemm_flow_takes(d) && flow_time(d) < *t ? GEMM_ROUTE_FLOW : shape;
}

int ecospa_gemm_route(const GemmDesc& d) {
  double t;
  int share;
  if (d.tile >= 50 && d.tile < 50 + GEMM_SHARE_NSHAPES && gemm_share_takes(d)) return GEMM_ROUTE_SHARE + d.tile - 50;
  const int route = tiled_route(d, &t);
  if (d.tile == 0 && route != GEMM_ROUTE_FLOW && gemm_share_takes(d) && share_plan(d, d.epi.kind, &share) < t + ring_cold(route, (d.K + 63) / 64)) return GEMM_ROUTE_SHARE + share;
  return route;
}

int ecospa_gemm(ecospa_ctx* ctx, const GemmDesc& d) {
  const int bad = gemm_check(d);
  if (bad) return bad;
  const int splits = d.splits > 1 ? d.splits : 1;
  if (d.dtype == ECOSPA_BF16) {
    const bool prof = prof_begin(ctx);
    const int k_chunk = ring_chunk(d, splits), shape = ecospa_gemm_route(d);
    hipError_t le;
    if (shape >= GEMM_ROUTE_SHARE) le = gemm_share_launch_nt(ctx, d, shape - GEMM_ROUTE_SHARE);
    else if (shape == GEMM_ROUTE_FLOW) le = d.trans_a ? gemm_flow_launch_tt(ctx, d) : gemm_flow_launch_nt(ctx, d);
    else if (d.trans_a && d.trans_b) le = gemm_ring_launch_tt(ctx, d, shape, k_chunk);
    else if (d.trans_a || d.trans_b) le = gemm_ring_launch_mixed(ctx, d, shape, k_chunk);
    else le = gemm_ring_launch_nt(ctx, d, shape, k_chunk);
    if (le != hipSuccess) return hip_fail(ctx, le, "gemm launch");
    if (prof) prof_end(ctx, 2.0 * d.M * d.N * d.K);
    ECOSPA_CHECK_LAUNCH(ctx, "gemm_bf16_ring_kernel");
  } else {
    if (!d.trans_a && !d.trans_b) launch_f32<false, false>(ctx, d, splits);
    else if (!d.trans_a) launch_f32<false, true>(ctx, d, splits);
    else if (d.trans_b) launch_f32<true, true>(ctx, d, splits);
    else launch_f32<true, false>(ctx, d, splits);
    ECOSPA_CHECK_LAUNCH(ctx, "gemm_f32_kernel");
  }
  if (splits > 1 && !d.defer_reduce) return ecospa_gemm_reduce(ctx, d);
  return ECOSPA_OK;
}

// Byte ranges that a descriptor reads and writes.
struct GemmRange {
  uintptr_t lo, hi;
  bool apart(const GemmRange& o) const { return hi <= o.lo || o.hi <= lo; }
};
static GemmRange mat_range(const void* p, long long rows, long long ld, long long cols, int bytes) {
  const uintptr_t lo = reinterpret_cast<uintptr_t>(p);
  return {lo, p ? lo + static_cast<uintptr_t>(((rows - 1) * ld + cols) * bytes) : lo};
}
// Neither reads what the other writes, nor do they write the same (a caller may pass one buffer for an input and a gradient: then they
// have to run in order).
static bool gemm_independent(const GemmDesc& w, const GemmDesc& x) {
  const int es = static_cast<int>(dtype_size(w.dtype)), splits = w.splits > 1 ? w.splits : 1;
  const GemmRange in_w[2] = {mat_range(w.A, w.K, w.lda, w.M, es), mat_range(w.B, w.K, w.ldb, w.N, es)};
  const GemmRange in_x[2] = {x.trans_a ? mat_range(x.A, x.K, x.lda, x.M, es) : mat_range(x.A, x.M, x.lda, x.K, es),
                             x.trans_b ? mat_range(x.B, x.K, x.ldb, x.N, es) : mat_range(x.B, x.N, x.ldb, x.K, es)};
  const long long wide = x.epi.kind == EPI_DSWIGLU ? 2ll * x.N : x.N;
  const GemmRange out_x = mat_range(x.epi.c, x.M, x.epi.ldc, wide, es), side_x = mat_range(x.epi.h, x.M, x.epi.ldh, wide, es);
  const GemmRange out_w[2] = {splits > 1 ? mat_range(w.partial, splits, static_cast<long long>(w.M) * w.N, static_cast<long long>(w.M) * w.N, 4)
                                         : mat_range(w.epi.c, w.M, w.epi.ldc, w.N, es),
                              mat_range(w.colsum, w.colsum ? ecospa_gemm_colsum_rows(w) : 1, w.M, w.M, 4)};
  bool ok = true;
  for (int i = 0; i < 2; ++i) {
    ok = ok && out_x.apart(in_w[i]) && out_x.apart(out_w[i]) && side_x.apart(out_w[i]);
    for (int j = 0; j < 2; ++j) ok = ok && out_w[i].apart(in_x[j]);
  }
  return ok;
}

// Whether one launch is the better way for two contractions of these shapes: where together they leave a good part of a round of compute
// units (64 of 512) to nobody, which the other's tiles then take.  Forward and backward of a 384-wide layer on 12017 tokens (252 + 189, 96
// + 188 and 216 + 189 workgroups) 251 -> 242 us; pairs of full rounds gain nothing (256 + 256 workgroups: -0.6 .. +5 us, the tiles
// that share operands no longer run side by side).  200 pairs of random sizes that the rule takes, on 15 of the 16 shape pairs: 1.18x in the geometric
// mean against the two launches one behind the other (1.29x with 64x128 weight-gradient tiles, 1.01 - 1.10x with larger ones), one slower (0.974x).
static bool pair_pays(const GemmDesc& w, int splits, int ws, const GemmDesc& x, int xs) {
  const auto idle = [](const GemmDesc& d, int sp, const RingShape& r) {
    const long long n = static_cast<long long>((d.M + r.bm - 1) / r.bm) * ((d.N + r.bn - 1) / r.bn) * sp;
    return static_cast<int>((256 - n % 256) % 256);
  };
  return idle(w, splits, RING_SHAPES[ws]) + idle(x, 1, RING_SHAPES[xs]) >= 64;
}

int ecospa_gemm_pair_route(const GemmDesc& w, const GemmDesc& x, int* w_shape, int* x_shape) {
  *w_shape = *x_shape = -1;
  if (w.dtype != x.dtype || !w.trans_a || !w.trans_b || x.trans_a || x.splits > 1 || !gemm_independent(w, x)) return GEMM_PAIR_NONE;
  const int splits = w.splits > 1 ? w.splits : 1;
  if (w.dtype == ECOSPA_BF16) {
    if (x.trans_b || x.epi.kind != EPI_STORE || (splits > 1 && !w.defer_reduce) || ring_wide(w) || ring_wide(x)) return GEMM_PAIR_NONE;
    // x on its tiles of the ring kernel - but not where so few tokens would have it split along K, and it runs by itself with K shared out
    if (ecospa_gemm_shares_k(x) && ecospa_gemm_token_splits(x.M, x.N, x.K) > 1) return GEMM_PAIR_NONE;
    double t;
    const int ws = *w_shape = ecospa_gemm_route(w), xs = *x_shape = tiled_route(x, &t);
    if (ws == GEMM_ROUTE_FLOW || xs == GEMM_ROUTE_FLOW) return GEMM_PAIR_NONE;
    return RING_SHAPES[ws].bn == 128 && ((GEMM_PAIR_X >> xs) & 1) && pair_pays(w, splits, ws, x, xs) ? GEMM_PAIR_BF16 : GEMM_PAIR_NONE;
  }
  // fp32: while both are on tiles that share out K, that is bound by the latency of their launches (forward and backward of 512 tokens,
  // 256 -> 512 units: 71.4 -> 57.4 us with two pairs and the bias gradients out of the weight gradients, eight launches instead of eleven)
  return splits == 1 && !f32_wide_tiles(w, 1) && !f32_wide_tiles(x, 1) ? GEMM_PAIR_F32 : GEMM_PAIR_NONE;
}

int ecospa_gemm_pair(ecospa_ctx* ctx, const GemmDesc& w, const GemmDesc& x, int x_first) {
  int rc;
  if ((rc = gemm_check(w)) || (rc = gemm_check(x))) return rc;
  int ws, xs;
  const int route = ecospa_gemm_pair_route(w, x, &ws, &xs);
  if (route == GEMM_PAIR_BF16) {
    const int k_chunk = ring_chunk(w, w.splits > 1 ? w.splits : 1), bm = RING_SHAPES[ws].bm;
    const bool prof = prof_begin(ctx);
    const hipError_t le = bm == 64 ? gemm_pair_launch_64(ctx, w, x, xs, k_chunk) : bm == 128 ? gemm_pair_launch_128(ctx, w, x, xs, k_chunk)
                        : bm == 192 ? gemm_pair_launch_192(ctx, w, x, xs, k_chunk) : gemm_pair_launch_256(ctx, w, x, xs, k_chunk);
    if (le != hipSuccess) return hip_fail(ctx, le, "gemm pair launch");
    if (prof) prof_end(ctx, 2.0 * w.M * w.N * w.K + 2.0 * x.M * x.N * x.K);
    ECOSPA_CHECK_LAUNCH(ctx, "gemm_bf16_pair_kernel");
    return ECOSPA_OK;
  }
  if (route == GEMM_PAIR_F32) {
    const int wn = (w.N + 31) / 32, xn = (x.N + 31) / 32, n_w = (w.M + 31) / 32 * wn, n_x = (x.M + 31) / 32 * xn;
    const auto kern = f32_few(n_w + n_x, true) ? (x.trans_b ? gemm_f32_pair_kernel<true, true> : gemm_f32_pair_kernel<false, true>)
                                               : (x.trans_b ? gemm_f32_pair_kernel<true, false> : gemm_f32_pair_kernel<false, false>);
    hipLaunchKernelGGL(kern, dim3(n_w + n_x), dim3(256), 0, ctx->stream, w, x, wn, n_w, xn);
    ECOSPA_CHECK_LAUNCH(ctx, "gemm_f32_pair_kernel");
    return ECOSPA_OK;
  }
  if ((rc = ecospa_gemm(ctx, x_first ? x : w))) return rc;
  return ecospa_gemm(ctx, x_first ? w : x);
}

int ecospa_gemm_reduce(ecospa_ctx* ctx, const GemmDesc& d) {
  if (d.splits <= 1) return ECOSPA_OK;
  if (!d.partial || (!d.epi.c && d.epi.kind != EPI_SWIGLU)) return ECOSPA_ERR_NULL;
  const long long tot = static_cast<long long>(d.M) * d.N;
  if (d.dtype == ECOSPA_BF16)
    hipLaunchKernelGGL(gemm_splitk_reduce_vec8_kernel, dim3(static_cast<unsigned>((tot / 8 + 255) / 256)), dim3(256), 0,
                       ctx->stream, d);
  else
    hipLaunchKernelGGL((gemm_splitk_reduce_kernel<float>), dim3(static_cast<unsigned>((tot + 255) / 256)), dim3(256), 0,
                       ctx->stream, d);
  ECOSPA_CHECK_LAUNCH(ctx, "gemm_splitk_reduce_kernel");
  return ECOSPA_OK;
}

// ---------------------------------------------------------------------------------------------
// batched tail of a backward pass: split-K reductions and bias-gradient column sums in one launch
// ---------------------------------------------------------------------------------------------
#define AUX_THREADS 1024

struct AuxBatchDev {
  AuxBatch b;
  int blk_begin[2 * AUX_MAX_JOBS + 1];   // column sums first (long dependent chains), then reductions
};

template <typename T>
__device__ __forceinline__ void aux_reduce_block(const GemmDesc& d, int blk) {
  const long long tot = static_cast<long long>(d.M) * d.N;
  if (sizeof(T) == 2) {      // 8 consecutive columns per thread (N is a multiple of 8)
    const long long e = (static_cast<long long>(blk) * AUX_THREADS + threadIdx.x) * 8;
    if (e >= tot) return;
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = 0.f;
    for (int z0 = 0; z0 < d.splits; z0 += 4) {     // four partials in flight, added in split order
      float4 lo[4], hi[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool on = z0 + q < d.splits;
        const float* p = d.partial + (on ? z0 + q : z0) * tot + e;
        lo[q] = *reinterpret_cast<const float4*>(p);
        hi[q] = *reinterpret_cast<const float4*>(p + 4);
        if (!on) lo[q] = hi[q] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        v[0] += lo[q].x; v[1] += lo[q].y; v[2] += lo[q].z; v[3] += lo[q].w;
        v[4] += hi[q].x; v[5] += hi[q].y; v[6] += hi[q].z; v[7] += hi[q].w;
      }
    }
    epi_apply_vec8(d.epi, static_cast<int>(e / d.N), static_cast<int>(e % d.N), v);
  } else {
    const long long e = static_cast<long long>(blk) * AUX_THREADS + threadIdx.x;
    if (e >= tot) return;
    float s = 0.f;
    for (int z = 0; z < d.splits; ++z) s += d.partial[z * tot + e];
    epi_apply<T>(d.epi, static_cast<int>(e / d.N), static_cast<int>(e % d.N), s);
  }
}

// One workgroup sums a strip of AUX_LANES x (16 bytes of columns) over all M rows: the row slots
// (AUX_THREADS / AUX_LANES of them) walk down the rows with 16-byte loads, several in flight, then
// the slots are added in a fixed order.  Narrow strips (a quarter of a 128-byte line) give enough
// workgroups to hide the latency; the four strips of a line are mapped to workgroup ids that differ
// by 8, 16 and 24, i.e. to the same XCD, so that the line is fetched into one L2 only.
#define AUX_LANES 2
template <typename T>
__device__ __forceinline__ void aux_colsum_block(const AuxColsum& c, int blk, float* lds, bool out_bf16) {
  static_assert(AUX_LANES == 2, "four strips of AUX_LANES x 16 bytes make one 128-byte line");
  constexpr int V = 16 / sizeof(T);          // columns per lane
  constexpr int W = AUX_LANES * V;           // strip width
  constexpr int SLOTS = AUX_THREADS / AUX_LANES;
  const T* __restrict__ X = static_cast<const T*>(c.X);
  const int slot = threadIdx.x / AUX_LANES, ln = threadIdx.x % AUX_LANES;
  {   // blk -> strip: workgroup ids are dealt round-robin to the 8 XCDs (job ranges start at multiples of 8)
    const int xcd = blk & 7, t = blk >> 3;
    blk = (((t >> 2) * 8 + xcd) << 2) + (t & 3);
  }
  if (blk * W >= c.N) return;     // padding of the range (whole workgroup)
  const int col0 = blk * W + ln * V;
  float acc[V];
#pragma unroll
  for (int i = 0; i < V; ++i) acc[i] = 0.f;
  const bool vec_ok = (c.ldx % V == 0) && ((reinterpret_cast<uintptr_t>(X) & 15u) == 0) && col0 + V <= c.N;
  if (vec_ok) {
    for (int r0 = slot; r0 < c.M; r0 += 8 * SLOTS) {
      uint4 u[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int r = r0 + q * SLOTS;
        u[q] = r < c.M ? *reinterpret_cast<const uint4*>(X + static_cast<long long>(r) * c.ldx + col0) : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        if (sizeof(T) == 2) {
          const uint32_t w[4] = {u[q].x, u[q].y, u[q].z, u[q].w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            acc[(2 * i) % V] += __uint_as_float(w[i] << 16);
            acc[(2 * i + 1) % V] += __uint_as_float(w[i] & 0xffff0000u);
          }
        } else {
          acc[0] += __uint_as_float(u[q].x); acc[1 % V] += __uint_as_float(u[q].y);
          acc[2 % V] += __uint_as_float(u[q].z); acc[3 % V] += __uint_as_float(u[q].w);
        }
      }
    }
  } else {
    for (int r = slot; r < c.M; r += SLOTS)
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (col0 + i < c.N) acc[i] += load_f32<T>(X + static_cast<long long>(r) * c.ldx + col0 + i);
  }
#pragma unroll
  for (int i = 0; i < V; ++i) lds[slot * (W + 1) + ln * V + i] = acc[i];
  __syncthreads();
  // W columns x 64 groups of SLOTS / 64 slots, then the 64 group sums by one wavefront per column
  constexpr int GROUPS = 64, PER = SLOTS / GROUPS;
  float part = 0.f;
  const int colw = threadIdx.x / GROUPS, grp = threadIdx.x % GROUPS;     // AUX_THREADS == W * 64 for bf16
  if (colw < W) {
    for (int k = 0; k < PER; ++k) part += lds[(grp * PER + k) * (W + 1) + colw];
  }
  part = wave_sum(part);     // lanes of a wavefront = the 64 groups of one column; fixed order
  if (colw < W && grp == 0) {
    const int col = blk * W + colw;
    if (col < c.N) {
      if (out_bf16) store_f32<bf16_t>(static_cast<bf16_t*>(c.out) + col, part);
      else store_f32<float>(static_cast<float*>(c.out) + col, part);
    }
  }
}

__global__ __launch_bounds__(AUX_THREADS) void bwd_aux_kernel(const AuxBatchDev a) {
  __shared__ float lds[(AUX_THREADS / AUX_LANES) * (AUX_LANES * 8 + 1)];
  const int blk = blockIdx.x;
  int j = 0;
  while (blk >= a.blk_begin[j + 1]) ++j;     // blk_begin[n_jobs] = grid size
  const int local = blk - a.blk_begin[j];
  if (j < a.b.n_colsum) {
    const AuxColsum& c = a.b.colsum[j];
    const bool out_bf16 = (c.out_dtype ? c.out_dtype : c.dtype) == ECOSPA_BF16;
    if (c.dtype == ECOSPA_BF16) aux_colsum_block<bf16_t>(c, local, lds, out_bf16);
    else aux_colsum_block<float>(c, local, lds, out_bf16);
  } else {
    const GemmDesc& d = a.b.reduce[j - a.b.n_colsum];
    if (d.dtype == ECOSPA_BF16) aux_reduce_block<bf16_t>(d, local);
    else aux_reduce_block<float>(d, local);
  }
}

int ecospa_aux_launch(ecospa_ctx* ctx, const AuxBatch& b) {
  if (b.n_reduce < 0 || b.n_reduce > AUX_MAX_JOBS || b.n_colsum < 0 || b.n_colsum > AUX_MAX_JOBS) return ECOSPA_ERR_SHAPE;
  AuxBatchDev a;
  memset(&a, 0, sizeof(a));
  a.b = b;
  long long blk = 0;
  int j = 0;
  for (int i = 0; i < b.n_colsum; ++i, ++j) {
    const AuxColsum& c = b.colsum[i];
    if (!c.X || !c.out) return ECOSPA_ERR_NULL;
    if (!dtype_ok(c.dtype) || c.M < 1 || c.N < 1) return ECOSPA_ERR_SHAPE;
    const int line = 4 * AUX_LANES * (c.dtype == ECOSPA_BF16 ? 8 : 4);   // columns of four strips
    a.blk_begin[j] = static_cast<int>(blk);                               // a multiple of 32: starts on XCD 0
    blk += ((c.N + line - 1) / line + 7) / 8 * 32;                        // 8 lines x 4 strips at a time
  }
  for (int i = 0; i < b.n_reduce; ++i, ++j) {
    const GemmDesc& d = b.reduce[i];
    if (d.splits <= 1 || !d.partial || (!d.epi.c && d.epi.kind != EPI_SWIGLU)) return ECOSPA_ERR_NULL;
    if (!dtype_ok(d.dtype)) return ECOSPA_ERR_DTYPE;
    a.blk_begin[j] = static_cast<int>(blk);
    const long long items = static_cast<long long>(d.M) * d.N / (d.dtype == ECOSPA_BF16 ? 8 : 1);
    blk += (items + AUX_THREADS - 1) / AUX_THREADS;
  }
  if (j == 0) return ECOSPA_OK;
  if (blk > (1ll << 30)) return ECOSPA_ERR_SHAPE;
  for (int q = j; q <= 2 * AUX_MAX_JOBS; ++q) a.blk_begin[q] = static_cast<int>(blk);
  hipLaunchKernelGGL(bwd_aux_kernel, dim3(static_cast<unsigned>(blk)), dim3(AUX_THREADS), 0, ctx->stream, a);
  ECOSPA_CHECK_LAUNCH(ctx, "bwd_aux_kernel");
  return ECOSPA_OK;
}
