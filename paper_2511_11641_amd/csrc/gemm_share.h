// The bf16 contraction kernel of few tokens, x W^T on one round of narrow tiles (not part of the C ABI).
//
// What bounds such a launch is how soon its operands arrive: an output of 61 rows has 48 tiles of 64x64 for 256 compute units, and each of
// them a chain of K / 64 slabs.  Splitting K over workgroups fills the chip but sends partial sums through memory to a second launch (3 us and more).
// Here narrow tiles fill it, down to 32x16, and what a narrow tile lacks in products per byte does not matter at this size; the chain is
// shared out: every wavefront of a workgroup computes the whole BM x BN tile over its own units of 64 k, dealt round the W wavefronts.  It
// streams them global -> LDS into D buffers of its own (128 bytes of a row at a time: 64 are 10 % slower), so the main loop has no barrier, and
// 128 - 160 KB per compute unit are on their way from the start where K has a unit for every buffer (64 W D: from 1536 on for 32x16, 768 for 64x32).  The W partial tiles meet in LDS at the end and are added in wavefront order.
//
// Weights from memory, kernel with K split over workgroups (or unsplit) -> this one, us: 61x3072x2048 10.6 -> 7.5 (32x32), 61x2048x1024 6.3 -> 3.9
// (32x16), 61x5504x2048 with SwiGLU 13.2 -> 10.4 (64x32), 61x2048x2752 11.4 -> 7.4, 17x2048x2752 9.9 -> 6.6, 200x2048x2752 13.4 -> 10.3, 512x768x768
// 5.3 -> 4.9.  Not for tiles as large as 64x64: a wavefront's first unit then only lands with everyone's, and 1024x1024x512 takes 5.9 us
// against 4.9 on 64x64 tiles whose wavefronts share every slab.
#pragma once
#include "gemm_ring.h"

template <int BM, int BN, int W, int D>
struct ShareTile {
  static constexpr int FM = BM / 16, FN = BN / 16, PA = BM / 8, PB = BN / 8, PER = PA + PB;
  static constexpr int UNIT = (BM + BN) * 128;                                                 // bytes of a unit of both operands
  static constexpr int AREA = D * UNIT > BM * BN * 4 ? D * UNIT : BM * BN * 4;                 // LDS of a wavefront: its units, then its partial tile
  static constexpr int PAIRS = FM * FN / 2, PPW = PAIRS > W ? PAIRS / W : 1;                   // pairs of 16x16 blocks; how many a wavefront finishes
  static_assert(W * AREA <= 160 * 1024, "LDS of a compute unit");
  static_assert(PAIRS % PPW == 0 && (FN % 2 == 0 || FN == 1) && (FN > 1 || FM % 2 == 0), "whole pairs");
  static_assert(PER * D < 64, "vmcnt range");
};

template <int N> __device__ __forceinline__ void share_wait_vm() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(ring_waitcnt(N, false));
  asm volatile("" ::: "memory");
}

template <int BM, int BN, int W, int D>
__global__ __launch_bounds__(W * 64) __attribute__((amdgpu_waves_per_eu(W / 4, W / 4)))
void gemm_bf16_share_kernel(const RingGrid w, const GemmDesc d) {
  typedef ShareTile<BM, BN, W, D> S;
  constexpr int FM = S::FM, FN = S::FN, PA = S::PA, PB = S::PB, PER = S::PER, UNIT = S::UNIT;
  extern __shared__ __attribute__((aligned(16))) bf16_t lds[];
  const int block = blockIdx.x, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;

  int zsplit, tile_row, tile_col;
  ring_place(w, block, false, zsplit, tile_row, tile_col);
  const int m0 = tile_row * BM, n0 = tile_col * BN;

  // units of this wavefront: wave, wave + W, ..; unit 0 takes the remainder of K (kv of its 64 k)
  const int units = (d.K + 63) >> 6, kv = d.K - (units - 1) * 64;
  const int n = units > wave ? (units - wave + W - 1) / W : 0;
  const int k_own = wave == 0 ? 0 : kv + (wave - 1) * 64;
  const char* pa = reinterpret_cast<const char*>(static_cast<const bf16_t*>(d.A) + static_cast<long long>(m0) * d.lda + k_own);
  const char* pb = reinterpret_cast<const char*>(static_cast<const bf16_t*>(d.B) + static_cast<long long>(n0) * d.ldb + k_own);
  const bool part = wave == 0 && kv < 64;
  unsigned oa[PA], ob[PB];
  {
    const int r = lane >> 3, k = ((lane & 7) ^ (lane >> 3)) * 8;       // chunk ^ (row % 8): the fragment reads of 16 rows then meet no bank twice
    const unsigned lda = static_cast<unsigned>(d.lda), ldb = static_cast<unsigned>(d.ldb);
#pragma unroll
    for (int i = 0; i < PA; ++i) oa[i] = (static_cast<unsigned>(min(i * 8 + r, d.M - 1 - m0)) * lda + k) * 2u;      // rows beyond the matrix repeat its last one
#pragma unroll
    for (int i = 0; i < PB; ++i) ob[i] = (static_cast<unsigned>(min(i * 8 + r, d.N - 1 - n0)) * ldb + k) * 2u;
  }
  lds_bf16_t* const my = (lds_bf16_t*)lds + wave * (S::AREA / 2);
  auto issue = [&](int buf, unsigned back) __attribute__((always_inline)) {
    lds_bf16_t* const dst = my + buf * (UNIT / 2);
#pragma unroll
    for (int i = 0; i < PA; ++i) __builtin_amdgcn_global_load_lds(reinterpret_cast<const void*>(pa + (oa[i] - back)), dst + i * 512, 16, 0, 0);
#pragma unroll
    for (int i = 0; i < PB; ++i) __builtin_amdgcn_global_load_lds(reinterpret_cast<const void*>(pb + (ob[i] - back)), dst + (PA + i) * 512, 16, 0, 0);
    pa += W * 128;
    pb += W * 128;
  };
  if (n > 0) {
    issue(0, part ? static_cast<unsigned>(max(((lane & 7) ^ (lane >> 3)) * 8 + 8 - kv, 0)) * 2u : 0u);
    if (part) { pa -= (64 - kv) * 2; pb -= (64 - kv) * 2; }
  }

  // What the epilogue reads besides the sums, asked for now: bias and side inputs of the groups of 8 columns that this lane finishes.
  constexpr int PPW = S::PPW;
  auto place = [&](int q, int& m, int& c) __attribute__((always_inline)) {
    const int p = wave * PPW + q;
    if constexpr (FN > 1) {
      m = m0 + p / (FN / 2) * 16 + l16;
      c = n0 + p % (FN / 2) * 32 + 16 * (g & 1) + 8 * (g >> 1);
    } else {
      m = m0 + (2 * p + (g & 1)) * 16 + l16;
      c = n0 + 8 * (g >> 1);
    }
  };
  const bool finishes = wave * PPW < S::PAIRS, has_bias = d.epi.bias != nullptr && d.epi.kind != EPI_DACT && d.epi.kind != EPI_DSWIGLU;
  uint4 braw[PPW];
  EpiSide side[PPW];
  if (finishes) {
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      int m, c;
      place(q, m, c);
      m = min(m, d.M - 1);
      c = min(c, d.N - 8);
      if (has_bias) braw[q] = *reinterpret_cast<const uint4*>(static_cast<const bf16_t*>(d.epi.bias) + c);
      if (d.epi.kind == EPI_ROPE) epi_side_load_k<EPI_ROPE>(d.epi, m, c, side[q]);
      else if (d.epi.kind == EPI_DACT) epi_side_load_k<EPI_DACT>(d.epi, m, c, side[q]);
      else if (d.epi.kind == EPI_DSWIGLU) epi_side_load_k<EPI_DSWIGLU>(d.epi, m, c, side[q]);
    }
  }
  asm volatile("" ::: "memory");
#pragma unroll
  for (int j = 1; j < D; ++j)
    if (j < n) issue(j, 0u);

  ring_f4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = ring_f4{0.f, 0.f, 0.f, 0.f};
  unsigned fr[2];        // fragment reads: row l16, 16-byte chunk 4 s + g
#pragma unroll
  for (int s = 0; s < 2; ++s) fr[s] = static_cast<unsigned>(reinterpret_cast<uintptr_t>(my)) + 2 * (l16 * 64 + (((4 * s + g) ^ (l16 & 7)) << 3));

  auto unit = [&](auto left_, int buf, bool first, bool more) __attribute__((always_inline)) {
    constexpr int left = decltype(left_)::value;      // loads that may still be under way: those of the units behind this one
    share_wait_vm<left>();
    ring_u4 fa[2][FM], fb[2][FN];
    ring_for<0, 2>([&](auto s_) __attribute__((always_inline)) {
      constexpr int s = decltype(s_)::value;
      const unsigned ad = fr[s] + buf * UNIT;
      ring_for<0, FM>([&](auto i_) __attribute__((always_inline)) {
        constexpr int i = decltype(i_)::value;
        ring_u4& r = fa[s][i];
        const unsigned at = ad;
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(at), "n"(i * 2048) : "memory");
      });
      ring_for<0, FN>([&](auto j_) __attribute__((always_inline)) {
        constexpr int j = decltype(j_)::value;
        ring_u4& r = fb[s][j];
        const unsigned at = ad;
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(at), "n"(BM * 128 + j * 2048) : "memory");
      });
    });
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int i = 0; i < FM; ++i) asm volatile("" : "+v"(fa[s][i]));
#pragma unroll
      for (int j = 0; j < FN; ++j) asm volatile("" : "+v"(fb[s][j]));
    }
    __builtin_amdgcn_sched_barrier(0);
    if (more) issue(buf, 0u);
    if (first && part) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const bool in = 32 * s + 8 * g < kv;
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[s][i] = in ? fa[s][i] : ring_u4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[s][j] = in ? fb[s][j] : ring_u4{0u, 0u, 0u, 0u};
      }
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fb[s][j]), __builtin_bit_cast(bf16x8_t, fa[s][i]), acc[i][j], 0, 0, 0);
  };
  int i = 0, buf = 0;
  auto next = [&]() __attribute__((always_inline)) { ++i; buf = buf + 1 == D ? 0 : buf + 1; };
#pragma unroll 1
  for (; n - i > D; next()) unit(ring_ic<PER * (D - 1)>{}, buf, i == 0, true);
  ring_for<0, D>([&](auto t_) __attribute__((always_inline)) {
    constexpr int t = D - decltype(t_)::value;        // units left
    if (n - i >= t) {
      unit(ring_ic<PER * (t - 1)>{}, buf, i == 0, false);
      next();
    }
  });

  // Partial tiles: block (i, j) of a wavefront is 1 KB, lane by lane, in its own LDS.
  float4* const mine = reinterpret_cast<float4*>(reinterpret_cast<char*>(lds) + wave * S::AREA) + lane;
#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < FN; ++b) mine[(a * FN + b) * 64] = make_float4(acc[a][b][0], acc[a][b][1], acc[a][b][2], acc[a][b][3]);
  __syncthreads();
  if (!finishes) return;
  const char* const from = reinterpret_cast<const char*>(lds) + wave * (PPW * 2048) + lane * 16;
  epi_dispatch(d.epi.kind, [&](auto kind_) __attribute__((always_inline)) {
    constexpr int KIND = decltype(kind_)::value;
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      float4 x[W], y[W];
#pragma unroll
      for (int z = 0; z < W; ++z) {
        x[z] = *reinterpret_cast<const float4*>(from + z * S::AREA + q * 2048);
        y[z] = *reinterpret_cast<const float4*>(from + z * S::AREA + q * 2048 + 1024);
      }
#pragma unroll
      for (int z = 1; z < W; ++z) {
        x[0].x += x[z].x; x[0].y += x[z].y; x[0].z += x[z].z; x[0].w += x[z].w;
        y[0].x += y[z].x; y[0].y += y[z].y; y[0].z += y[z].z; y[0].w += y[z].w;
      }
      const float xs[4] = {x[0].x, x[0].y, x[0].z, x[0].w}, ys[4] = {y[0].x, y[0].y, y[0].z, y[0].w};
      float v[8], b[8];
#pragma unroll
      for (int r = 0; r < 4; ++r) {       // odd and even lane groups swap: a lane then holds 8 consecutive columns
        const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(xs[r]), __float_as_uint(ys[r]), false, false);
        v[r] = __uint_as_float(p[0]);
        v[4 + r] = __uint_as_float(p[1]);
      }
      int m, c;
      place(q, m, c);
      if (has_bias) unpack8(braw[q], b);
      if (m < d.M && c < d.N) epi_apply_vec8_k<KIND>(d.epi, m, c, v, has_bias, b, side[q]);
    }
  });
}

template <int BM, int BN, int W, int D>
static hipError_t share_launch_shape(ecospa_ctx* ctx, const GemmDesc& d) {
  const RingGrid w = gemm_ring_grid(d.M, d.N, BM, BN, 1, 0);
  constexpr int lds_bytes = W * ShareTile<BM, BN, W, D>::AREA;
  auto kern = gemm_bf16_share_kernel<BM, BN, W, D>;
  static LdsAttrOnce attr_once;
  if (lds_bytes > 64 * 1024) {
    const hipError_t e = attr_once.ensure(reinterpret_cast<const void*>(kern), lds_bytes);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(w.tiles), dim3(W * 64), lds_bytes, ctx->stream, w, d);
  return hipGetLastError();
}
