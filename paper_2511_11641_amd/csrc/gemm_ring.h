// The bf16 contraction kernel (not part of the C ABI).
//
// C[m, n] = sum_k A(m, k) B(n, k), either operand K-contiguous ([rows][K]) or K-slow ([K][rows]): x W^T, dY W and dY^T X are
// the same code.  A workgroup of four wavefronts, one per SIMD, owns a BM x BN tile of C (a wavefront BM/2 x BN/2, its
// accumulators in AGPRs).  Operand slabs of 64 k travel global -> LDS with direct loads (no registers in between) into a ring
// of NS buffers.
//
// What bounds it, and what follows from that (figures: N(0,1) operands, this GPU):
//   * Power.  The matrix units alone sustain 1.82 PFLOP/s with v_mfma_f32_32x32x16_bf16 and 2.10 PFLOP/s with
//     v_mfma_f32_16x16x32_bf16 (same issue rate, half the accumulator traffic per product), so the 16x16x32 form is used.
//   * Exposed LDS latency.  LDS delivers 256 bytes per clock and compute unit; a loop with one 16-byte fragment read per 32 cycles of
//     MFMA keeps a lone wavefront's matrix unit 96 % busy as long as no wait follows a read closely.  So the fragments of a 32-wide
//     k step are held twice: the reads of the next step are dealt over the first three quarters of the MFMAs of this one
//     (one wait per step, for reads that are at least a quarter step old; dealt over a quarter of them the K-slow form is 12 % slower).
//   * The compiler's own waits.  It cannot tell the ring buffers apart and waits for every direct load in flight before a transposing
//     LDS read; the reads are therefore inline assembly, with the waits written out.  The products are inline assembly where the
//     accumulators fill the AGPRs, or copies between the two register files appear in the loop.
// Against the kernels it replaced (direct loads with compiler-placed waits for x W^T, a register-staged one for dY^T X):
// 4096x2048x2752 x W^T 59 -> 45 us (256x128), dY^T X 2048x2752x4096 59.5 -> 44.6 us, 5504x2048x4096 99 -> 76 us.
// dY^T X 2048x1024x4096 takes 33 us as it did, on 64x128 tiles unsplit (128x128, K split in two, operands warm: 22 us).
//
// K need not be a multiple of anything in the K-slow forms (8 in the K-contiguous ones): the FIRST slab takes the remainder,
// with clamped addresses, and its k beyond the remainder are zeroed in LDS before the loop starts.
//
// LDS layout: 16-byte chunks, XOR-swizzled on the GLOBAL side of the direct load (the lane that owns a physical chunk fetches the
// logical chunk that maps there):
//   K-contiguous tile [rows][64]:  chunk ^ (row % 8): the lanes of an access fall on different banks (no conflicts counted)
//   K-slow tile [64][rows]:        the transposing reads of half a wavefront (32 lanes, one pass over the 64 banks) take 32 bytes of eight
//                                  rows, k .. k + 3 and k + 8 .. k + 11.  Rows of 128 and 256 start at the same bank: chunk ^ 4 (k % 4) ^ 2 (k / 8 % 2)
//                                  puts the eight pieces on eight bank groups; rows of 64 and 192 start half-way round the banks for odd k: chunk ^ 2 (k / 2 % 2)
//                                  ^ 4 (k / 8 % 2), inside groups of eight chunks.  No conflicts counted either (with the rows k + 8 on the banks
//                                  of the rows k, 49-62 % of these launches' LDS cycles were conflicts: 768x384x12017 16.5 -> 14.3 us on 64x128,
//                                  2048x1024x8192 in two parts 41.7 -> 39.8 us on 128x128; launches on larger tiles, which power bounds, 0 - 2 %).
#pragma once
#include "gemm_epi.h"

#include <type_traits>

typedef __attribute__((address_space(3))) bf16_t lds_bf16_t;
typedef unsigned int ring_u4 __attribute__((ext_vector_type(4)));
typedef unsigned int ring_u2 __attribute__((ext_vector_type(2)));
typedef float ring_f4 __attribute__((ext_vector_type(4)));

#define RING_BK 64

template <int V> using ring_ic = std::integral_constant<int, V>;
template <int I, int N, typename F>
__device__ __forceinline__ void ring_for(F&& f) {
  if constexpr (I < N) {
    f(ring_ic<I>{});
    ring_for<I + 1, N>(f);
  }
}

// s_waitcnt immediate: at most vm direct loads in flight, LDS counter untouched or zero
__host__ __device__ constexpr int ring_waitcnt(int vm, bool lgkm0) {
  return (vm & 15) | ((vm >> 4) << 14) | (7 << 4) | ((lgkm0 ? 0 : 15) << 8);
}

template <int RT>
__device__ __forceinline__ int ring_ks_swz(int k) {
  return RT % 128 == 0 ? ((k & 3) << 2) | (((k >> 3) & 1) << 1) : (((k >> 3) & 1) << 2) | (((k >> 1) & 1) << 1);
}

// Direct loads of one operand tile of RT rows: PER instructions per slab and wavefront, each moving 64 x 16 bytes to consecutive LDS.
// Addresses are a wavefront-uniform base (scalar registers, advanced by scalar adds) plus a lane offset that never changes: 32 bits, or
// 64 (WIDE) for leading dimensions whose tiles reach over 4 GB.
template <bool WIDE> using ring_off = std::conditional_t<WIDE, unsigned long long, unsigned>;
template <int RT, bool KSLOW, bool WIDE>
struct RingLoads {
  static constexpr int PER = RT * RING_BK * 2 / 1024 / 4;
  static_assert(PER * 4096 == RT * RING_BK * 2, "whole load instructions per wavefront");
  const char* base;
  ring_off<WIDE> off[PER];
  long long step;        // bytes per slab
  // first slab: kv (1 .. 64) of k, loaded here into `tile`; single: there is no other slab (the offsets then stay the clamped ones)
  __device__ __forceinline__ void init(const bf16_t* mat, long long ld, int r0, int R, int k0, int kv, bool single, bf16_t* tile) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lds_bf16_t* const dst = (lds_bf16_t*)tile + wave * PER * 512;
    base = reinterpret_cast<const char*>(KSLOW ? mat + static_cast<long long>(k0) * ld + r0 : mat + static_cast<long long>(r0) * ld + k0);
    const int last = R - r0 - (KSLOW ? 8 : 1);       // rows beyond the matrix repeat its last ones (never stored)
    const ring_off<WIDE> ldo = static_cast<ring_off<WIDE>>(ld);
    ring_off<WIDE> back[PER];        // how far the clamped address of the first slab lies behind that of a whole one
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int p = (wave * PER + i) * 64 + lane;      // physical chunk of the tile
      if constexpr (!KSLOW) {
        const int k = ((lane & 7) ^ (lane >> 3)) * 8;
        off[i] = (static_cast<ring_off<WIDE>>(min(p / 8, last)) * ldo + static_cast<ring_off<WIDE>>(k)) * 2u;
        back[i] = static_cast<ring_off<WIDE>>(max(k + 8 - kv, 0)) * 2u;
      } else {
        const int k = p / (RT / 8);
        off[i] = (static_cast<ring_off<WIDE>>(k) * ldo + static_cast<ring_off<WIDE>>(min(((p % (RT / 8)) ^ ring_ks_swz<RT>(k)) * 8, last))) * 2u;
        back[i] = static_cast<ring_off<WIDE>>(max(k + 1 - kv, 0)) * ldo * 2u;
      }
    }
    if (kv == RING_BK) {
#pragma unroll
      for (int i = 0; i < PER; ++i) __builtin_amdgcn_global_load_lds(reinterpret_cast<const void*>(base + off[i]), dst + i * 512, 16, 0, 0);
    } else {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        __builtin_amdgcn_global_load_lds(reinterpret_cast<const void*>(base + (off[i] - back[i])), dst + i * 512, 16, 0, 0);
        if (single) off[i] -= back[i];
      }
    }
    if (!single) base += KSLOW ? static_cast<long long>(kv) * ld * 2 : kv * 2;
    step = KSLOW ? static_cast<long long>(RING_BK) * ld * 2 : RING_BK * 2;
  }
  // instruction i of a slab into `tile`; the last one moves the base on by `adv`: the step, or 0 once there is no further slab - the
  // last slab is then loaded again, into buffers that nobody reads any more, which keeps the loop free of branches
  __device__ __forceinline__ void issue(int i, lds_bf16_t* tile, long long adv) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    asm volatile("" : "+v"(off[i]));     // keeps the offset a lane register at the load
    __builtin_amdgcn_global_load_lds(reinterpret_cast<const void*>(base + off[i]), tile + (wave * PER + i) * 512, 16, 0, 0);
    if (i == PER - 1) base += adv;
  }
  // zeros for the k >= kv of a tile that holds kv of them
  __device__ __forceinline__ static void zero_tail(bf16_t* tile, int kv) {
    for (int p = threadIdx.x; p < RT * RING_BK / 8; p += 256) {
      const int k = KSLOW ? p / (RT / 8) : ((p % 8) ^ ((p / 8) & 7)) * 8;
      if (k >= kv) *reinterpret_cast<ring_u4*>(tile + p * 8) = ring_u4{0u, 0u, 0u, 0u};
    }
  }
};

// Fragment reads of one operand: fragment f (16 rows) of k step s, lane (l16, g): row l16, k = 32 s + 8 g .. + 7.
// K-slow: two transposing reads (4 k each); inside a group of 16 lanes, lane i addresses (k + i / 4, rows 4 (i % 4) ..+3) and
// receives row i of the group's four k.
template <int RT, bool KSLOW, int F>
struct RingFrags {
  static constexpr int NA = KSLOW ? F : 2;
  unsigned addr[NA];
  __device__ __forceinline__ void init(const bf16_t* tile, int row0) {
    const int lane = threadIdx.x & 63, g = lane >> 4, i = lane & 15;
    const unsigned t = static_cast<unsigned>(reinterpret_cast<uintptr_t>((const lds_bf16_t*)tile));
    if constexpr (!KSLOW) {
#pragma unroll
      for (int s = 0; s < NA; ++s) addr[s] = t + 2 * ((row0 + i) * RING_BK + (((4 * s + g) ^ ((row0 + i) & 7)) << 3));
    } else {
      const int k = 8 * g + (i >> 2);
#pragma unroll
      for (int f = 0; f < NA; ++f) {
        const int r = row0 + f * 16 + 4 * (i & 3);
        addr[f] = t + 2 * (k * RT + (((r >> 3) ^ ring_ks_swz<RT>(k)) << 3) + (r & 7));
      }
    }
  }
};
struct RingFrag { ring_u2 lo, hi; ring_u4 v; };     // K-slow: the two halves; K-contiguous: v
template <bool KS> __device__ __forceinline__ void ring_tie(RingFrag& r) {     // behind a wait: the values may be used from here on
  if constexpr (KS) asm volatile("" : "+v"(r.lo), "+v"(r.hi));
  else asm volatile("" : "+v"(r.v));
}
template <bool KS> __device__ __forceinline__ bf16x8_t ring_val(const RingFrag& r) {
  if constexpr (KS) {
    const ring_u4 v = {r.lo[0], r.lo[1], r.hi[0], r.hi[1]};
    return __builtin_bit_cast(bf16x8_t, v);
  } else {
    return __builtin_bit_cast(bf16x8_t, r.v);
  }
}
__device__ __forceinline__ void ring_mfma(ring_f4& c, const bf16x8_t& a, const bf16x8_t& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

// a / d with the inverse of d that RingGrid has beside it: the product's high half falls short by one at most
__device__ __forceinline__ int ring_div(int a, int d, unsigned inv, int& rest) {
  int q = static_cast<int>(__umulhi(static_cast<unsigned>(a), inv));
  rest = a - q * d;
  if (rest >= d) { ++q; rest -= d; }
  return q;
}

// Tile (row, column) and K split of workgroup `block`.
__device__ __forceinline__ void ring_place(const RingGrid& w, int block, bool split, int& zsplit, int& row, int& col) {
  const int xcd = block & 7;
  int id = xcd * w.per + min(xcd, w.more) + (block >> 3), in_band;
  zsplit = 0;
  if (split) zsplit = ring_div(id, w.tiles, w.tiles_inv, id);
  const int band = ring_div(id, w.band, w.band_inv, in_band);
  const bool last_band = band == w.last_band;
  col = ring_div(in_band, last_band ? w.last_rows : w.group, last_band ? w.last_inv : w.group_inv, row);
  row += band * w.group;
}

// One output tile (of one K split): that of workgroup `block` of the grid w.
// EPIS: bit mask of the epilogue kinds the instantiation carries; CS: column sums of a K-slow A (GemmDesc::colsum); WIDE: see ring_off.
template <int BM, int BN, int NS, bool TA, bool TB, bool CS, int EPIS, bool WIDE>
__device__ __forceinline__ void ring_tile(const GemmDesc& d, const RingGrid& w, int block) {
  constexpr int WTM = BM / 2, WTN = BN / 2, FM = WTM / 16, FN = WTN / 16, S = RING_BK / 32, NM = FM * FN, NR = FM + FN;
  constexpr int STAGE = (BM + BN) * RING_BK;
  static_assert(FN % 2 == 0, "the epilogue pairs column blocks");
  static_assert(!CS || TA, "column sums are of a K-slow A");
  extern __shared__ __attribute__((aligned(16))) bf16_t lds[];
  lds_bf16_t* lds3 = (lds_bf16_t*)lds;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = __builtin_amdgcn_readfirstlane(wave & 1);

  const int tiles_n = w.tiles_n;
  int zsplit, tile_row, tile_col;
  ring_place(w, block, d.splits > 1, zsplit, tile_row, tile_col);
  const int m0 = tile_row * BM, n0 = tile_col * BN;
  const int k_begin = zsplit * w.k_chunk;
  const int k_end = min(d.K, k_begin + w.k_chunk);
  const int nk = (k_end - k_begin + RING_BK - 1) / RING_BK;
  const int kv = (k_end - k_begin) - (nk - 1) * RING_BK;         // k of the first slab

  if (nk <= 0) {        // an empty split (more splits than slabs): its partial sums are zeros
    float* part = d.partial + static_cast<long long>(zsplit) * d.M * d.N;
    for (int e = threadIdx.x; e < BM * BN; e += 256) {
      const int m = m0 + e / BN, n = n0 + e % BN;
      if (m < d.M && n < d.N) part[static_cast<long long>(m) * d.N + n] = 0.f;
    }
    if constexpr (CS)
      for (int r = threadIdx.x; r < BM; r += 256)
        if (m0 + r < d.M) d.colsum[(static_cast<long long>(zsplit) * tiles_n + tile_col) * d.M + m0 + r] = 0.f;
    return;
  }

  ring_f4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
  // column sums: dot products with a pair of ones
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const bf16x2_t one = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
  float cs[CS ? FM : 1];
#pragma unroll
  for (int i = 0; i < (CS ? FM : 1); ++i) cs[i] = 0.f;

  RingLoads<BM, TA, WIDE> la;
  RingLoads<BN, TB, WIDE> lb;
  constexpr int PA = RingLoads<BM, TA, WIDE>::PER, PB = RingLoads<BN, TB, WIDE>::PER, LPW = PA + PB;
  static_assert(LPW * (NS - 1) < 64, "vmcnt range");
  la.init(static_cast<const bf16_t*>(d.A), d.lda, m0, d.M, k_begin, kv, nk == 1, lds);
  lb.init(static_cast<const bf16_t*>(d.B), d.ldb, n0, d.N, k_begin, kv, nk == 1, lds + BM * RING_BK);
  // A lane keeps its columns (see the epilogue) for every row: their bias is loaded once.  Tiles that leave registers for it ask for it here,
  // behind the first slab; asked for behind the loop it comes from memory while everything waits (stores out 0.75 -> 0.5 us behind the loop's end).
  const int l16 = lane & 15, g = lane >> 4, nw = n0 + wn * WTN + 16 * (g & 1) + 8 * (g >> 1);
  constexpr int JP = FN / 2;
  constexpr bool BIAS_EARLY = NM <= 24;      // (256x256 tiles: 32 x 1024 tokens, 1024 -> 1536 columns, 80 -> 87 us with the loop's registers so much fewer)
  uint4 braw[JP];
  const bool has_bias = d.splits <= 1 && d.epi.bias != nullptr && d.epi.kind != EPI_DACT && d.epi.kind != EPI_DSWIGLU;
  auto load_bias = [&]() __attribute__((always_inline)) {
    if (has_bias) {
#pragma unroll
      for (int j = 0; j < JP; ++j) braw[j] = *reinterpret_cast<const uint4*>(static_cast<const bf16_t*>(d.epi.bias) + min(nw + j * 32, d.N - 8));
    }
  };
  if constexpr (BIAS_EARLY) {
    load_bias();
    asm volatile("" ::: "memory");
  }
  auto issue = [&](auto q_, auto buf_, bool adv) __attribute__((always_inline)) {
    constexpr int q = decltype(q_)::value, buf = decltype(buf_)::value;
    if constexpr (q < PA) la.issue(q, lds3 + buf * STAGE, adv ? la.step : 0);
    else lb.issue(q - PA, lds3 + buf * STAGE + BM * RING_BK, adv ? lb.step : 0);
  };
  // Loads of a slab are dealt over the k steps behind the barrier that frees its buffer (in front of the last k step of a slab);
  // a ring of two needs them out in one step.
  constexpr int LSTEPS = NS == 2 ? S - 1 : S;
  constexpr int LPS = (LPW + LSTEPS - 1) / LSTEPS;
  ring_for<1, NS - 1>([&](auto p_) __attribute__((always_inline)) {
    ring_for<0, LPW>([&](auto q_) __attribute__((always_inline)) { issue(q_, p_, decltype(p_)::value + 1 < nk); });
  });
  RingFrags<BM, TA, FM> ra;
  RingFrags<BN, TB, FN> rb;
  ra.init(lds, wm * WTM);
  rb.init(lds + BM * RING_BK, wn * WTN);

  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(ring_waitcnt((NS - 2) * LPW, false));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  if (kv < RING_BK) {
    RingLoads<BM, TA, WIDE>::zero_tail(lds, kv);
    RingLoads<BN, TB, WIDE>::zero_tail(lds + BM * RING_BK, kv);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
  RingFrag fa[2][FM], fb[2][FN];
  // fragment read number f, in the order the products need them: a0, b0 .. bFN-1, a1 .. aFM-1
  auto rd = [&](auto set_, auto buf_, auto s_, auto f_) __attribute__((always_inline)) {
    constexpr int set = decltype(set_)::value, buf = decltype(buf_)::value, s = decltype(s_)::value, f = decltype(f_)::value;
    constexpr bool isb = f >= 1 && f <= FN;
    constexpr int i = f == 0 ? 0 : (isb ? f - 1 : f - FN);
    constexpr bool ks = isb ? TB : TA;
    constexpr int RT = isb ? BN : BM;
    constexpr int tot = buf * STAGE * 2 + (ks ? s * 32 * RT * 2 : i * 16 * RING_BK * 2);
    constexpr int imm = tot & 32767, big = tot - imm;
    RingFrag& r = isb ? fb[set][i] : fa[set][i];
    const unsigned ad = (isb ? rb.addr[ks ? i : s] : ra.addr[ks ? i : s]) + big;
    if constexpr (ks) {
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r.lo) : "v"(ad), "n"(imm));
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r.hi) : "v"(ad), "n"(imm + 4 * RT * 2));
    } else {
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r.v) : "v"(ad), "n"(imm));
    }
  };
  auto landed = [&](auto set_) __attribute__((always_inline)) {
    constexpr int set = decltype(set_)::value;
    ring_for<0, FM>([&](auto i_) __attribute__((always_inline)) { ring_tie<TA>(fa[set][decltype(i_)::value]); });
    ring_for<0, FN>([&](auto j_) __attribute__((always_inline)) { ring_tie<TB>(fb[set][decltype(j_)::value]); });
    __builtin_amdgcn_sched_barrier(0);
  };
  ring_for<0, NR>([&](auto f_) __attribute__((always_inline)) { rd(ring_ic<0>{}, ring_ic<0>{}, ring_ic<0>{}, f_); });
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  landed(ring_ic<0>{});

  // column sums: wavefront column wn of tile column j takes the slabs whose number is 2 j + wn modulo twice the tile columns
  int cs_next = 2 * tile_col + wn;
  constexpr int RSLOTS = NM * 3 / 4;        // the reads of the next k step go behind the first three quarters of this one's products
  auto slab = [&](auto buf_, int t) __attribute__((always_inline)) {
    constexpr int buf = decltype(buf_)::value;
    constexpr int buf_next = (buf + 1) % NS, buf_prev = (buf + NS - 1) % NS;
    const bool cs_now = CS && t == cs_next;
    if (CS && cs_now) cs_next += 2 * tiles_n;
    ring_for<0, S>([&](auto s_) __attribute__((always_inline)) {
      constexpr int s = decltype(s_)::value;
      constexpr int cur = s & 1, nxt = cur ^ 1;
      constexpr bool last = s + 1 == S;
      constexpr int ls = last ? 0 : s + 1;        // load step: 0 right behind the barrier
      constexpr int Q0 = ls * LPS < LPW ? ls * LPS : LPW, Q1 = (ls + 1) * LPS < LPW ? (ls + 1) * LPS : LPW, NQ = Q1 - Q0;
      const bool adv = t + (last ? NS + 1 : NS) < nk;
      if constexpr (CS) {
        if (cs_now) {
          ring_for<0, FM>([&](auto i_) __attribute__((always_inline)) {
            constexpr int i = decltype(i_)::value;
            const unsigned w[4] = {fa[cur][i].lo[0], fa[cur][i].lo[1], fa[cur][i].hi[0], fa[cur][i].hi[1]};
#pragma unroll
            for (int q = 0; q < 4; ++q) cs[i] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w[q]), one, cs[i], false);
          });
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      ring_for<0, NM>([&](auto m_) __attribute__((always_inline)) {
        constexpr int m = decltype(m_)::value, i = m / FN, j = m % FN;
        // B's fragment first: the accumulators then hold four consecutive columns of one row (see the epilogue)
        ring_mfma(acc[i][j], ring_val<TB>(fb[cur][j]), ring_val<TA>(fa[cur][i]));
        __builtin_amdgcn_sched_barrier(0);
        constexpr int R0 = m < RSLOTS ? m * NR / RSLOTS : NR, R1 = m < RSLOTS ? (m + 1) * NR / RSLOTS : NR;
        ring_for<R0, R1>([&](auto f_) __attribute__((always_inline)) {
          rd(ring_ic<nxt>{}, ring_ic<(last ? buf_next : buf)>{}, ring_ic<(last ? 0 : s + 1)>{}, f_);
        });
        ring_for<Q0 + m * NQ / NM, Q0 + (m + 1) * NQ / NM>([&](auto q_) __attribute__((always_inline)) { issue(q_, ring_ic<(last ? buf : buf_prev)>{}, adv); });
        __builtin_amdgcn_sched_barrier(0);
      });
      // The fragments of the next k step have landed.  The wait closes the step instead of opening the next one, so that no read is
      // under way where control flow splits or joins: the compiler may move values between registers there, and it does not know
      // that they are still being written.
      if constexpr (!last) {
        // and slab t + 1 as well (own loads: the wait; everyone's: the barrier); everyone holds the last fragments of slab t,
        // whose buffer is refilled from here on
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(ring_waitcnt((NS - 2) * LPW, true));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      } else {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
      landed(ring_ic<nxt>{});
    });
  };
  static_assert(S == 2, "the two fragment sets alternate over a slab");
  ring_for<0, (LPS < LPW ? LPS : LPW)>([&](auto q_) __attribute__((always_inline)) { issue(q_, ring_ic<NS - 1>{}, NS < nk); });
  int t = 0;
  for (; t + NS <= nk; t += NS)
    ring_for<0, NS>([&](auto b_) __attribute__((always_inline)) { slab(b_, t + decltype(b_)::value); });
  ring_for<0, NS - 1>([&](auto b_) __attribute__((always_inline)) {
    if (t + decltype(b_)::value < nk) slab(b_, t + decltype(b_)::value);
  });
  // the repeated loads are still on their way into LDS, the last products into their accumulators
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) asm volatile("" : "+a"(acc[i][j]));
  __builtin_amdgcn_sched_barrier(0);

  if constexpr (CS) {
    // lanes of one l16 hold the sums over different k; the two wavefront columns took different slabs
    __syncthreads();                            // everyone's loads have landed: LDS is free
    float* red = reinterpret_cast<float*>(lds);     // [2][BM]
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      float v = cs[i];
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      if (g == 0) red[wn * BM + wm * WTM + i * 16 + l16] = v;
    }
    __syncthreads();
    for (int r = threadIdx.x; r < BM; r += 256)
      if (m0 + r < d.M) d.colsum[(static_cast<long long>(zsplit) * tiles_n + tile_col) * d.M + m0 + r] = red[r] + red[BM + r];
  }

  // Epilogue straight from the accumulators.  acc[i][j] of lane (l16, g): row i * 16 + l16, columns j * 16 + 4 g + 0..3; two
  // neighbouring column blocks swap their odd and even lane groups, so that a lane holds 8 consecutive columns (16-byte stores,
  // 64 bytes per row and instruction; staging the tile through LDS instead costs 4 us more on a 256x256 tile).
  const int mw = m0 + wm * WTM + l16;
  auto vals = [&](auto i_, auto jp_, float (&v)[8]) __attribute__((always_inline)) {
    constexpr int i = decltype(i_)::value, jp = decltype(jp_)::value;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[i][2 * jp][r]), __float_as_uint(acc[i][2 * jp + 1][r]), false, false);
      v[r] = __uint_as_float(p[0]);
      v[4 + r] = __uint_as_float(p[1]);
    }
  };
  if (d.splits > 1) {
    float* part = d.partial + static_cast<long long>(zsplit) * d.M * d.N;
    ring_for<0, FM>([&](auto i_) __attribute__((always_inline)) {
      const int m = mw + decltype(i_)::value * 16;
      ring_for<0, JP>([&](auto jp_) __attribute__((always_inline)) {
        float v[8];
        vals(i_, jp_, v);
        const int n = nw + decltype(jp_)::value * 32;
        if (m < d.M && n < d.N) {
          float* p = part + static_cast<long long>(m) * d.N + n;
          *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
          *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
        }
      });
    });
    return;
  }
  if constexpr (!BIAS_EARLY) load_bias();
  auto add_bias = [&](int jp, float (&v)[8]) __attribute__((always_inline)) {
    if (has_bias) {
      float b[8];
      unpack8(braw[jp], b);
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] += b[q];
    }
  };
  // Addresses: a base per workgroup (scalar) plus lane offsets; lane rows beyond the matrix read its last row and store nothing.
  const bool cols_in = n0 + BN <= d.N;
  const int row_l = wm * WTM + l16, rows_in = d.M - m0, nl = nw - n0, n_last = d.N - 8 - n0;
  char* const cb = reinterpret_cast<char*>(static_cast<bf16_t*>(d.epi.c) + static_cast<long long>(m0) * d.epi.ldc + (d.epi.kind == EPI_DSWIGLU ? 2 * n0 : n0));
  typedef ring_off<WIDE> off_t;
  const off_t ldc2b = static_cast<off_t>(d.epi.ldc) * 2u;      // bytes per row of c
  if (d.epi.kind == EPI_STORE) {
    ring_for<0, FM>([&](auto i_) __attribute__((always_inline)) {
      constexpr int i = decltype(i_)::value;
      const int row = row_l + i * 16;
      const off_t off = static_cast<off_t>(row) * ldc2b + nl * 2;
      uint4 o[JP];
      ring_for<0, JP>([&](auto jp_) __attribute__((always_inline)) {
        float v[8];
        vals(i_, jp_, v);
        add_bias(decltype(jp_)::value, v);
        o[decltype(jp_)::value] = pack8(v);
      });
      if (row < rows_in) {
#pragma unroll
        for (int jp = 0; jp < JP; ++jp)
          if (cols_in || nl + jp * 32 <= n_last) *reinterpret_cast<uint4*>(cb + off + jp * 64) = o[jp];
      }
    });
    return;
  }
  // The other kinds: their arithmetic on up to 32 groups of 8 columns, unrolled, would be tens of kilobytes of instructions that
  // every wavefront fetches once (GELU with two outputs on 8192x2048x1024, 256x256 tiles: 72 us).  Instead the accumulators
  // are parked in LDS, each lane's own values in its own slots (no exchange, no barrier), and a loop over the row blocks takes
  // them back.  Up to four groups go straight from the registers: their code is short, and the barrier and the trip through LDS stood behind a
  // short loop (24-layer forward on 1024 tokens, one GELU contraction on 128x64 tiles per layer: 1468 -> 1457 us).  Not the tanh form of GELU,
  // whose code is long (tanhf has two branches): its derivative on 128x64 tiles, 1400x520x720: 14.2 us from the registers, 13.5 through LDS.
  constexpr int SLOT_ROWS = NS * (BM + BN) * RING_BK * 2 / 4 / (JP * 2048);      // row blocks that a wavefront's share of LDS holds
  constexpr int CH = SLOT_ROWS >= FM ? FM : FM / 2;
  static_assert(CH >= 1 && CH <= SLOT_ROWS && FM % CH == 0, "LDS holds a whole chunk");
  constexpr bool PARK = FM * JP > 4;
  const bool park = PARK || (d.epi.act == ECOSPA_ACT_GELU_TANH && (d.epi.kind == EPI_BIAS_ACT || d.epi.kind == EPI_ACT || d.epi.kind == EPI_DACT));
  if (park) __syncthreads();                  // everyone's loads have landed
  char* const slots = reinterpret_cast<char*>(lds) + wave * (CH * JP * 2048) + lane * 16;
  epi_dispatch(d.epi.kind, [&](auto kind_) __attribute__((always_inline)) {
    constexpr int KIND = decltype(kind_)::value;
    if constexpr (KIND != EPI_STORE && ((EPIS >> KIND) & 1)) {
      const char* const hb = reinterpret_cast<const char*>(static_cast<const bf16_t*>(d.epi.h) + static_cast<long long>(m0) * d.epi.ldh + (KIND == EPI_DSWIGLU ? 2 * n0 : n0));
      char* const c2b = reinterpret_cast<char*>(static_cast<bf16_t*>(d.epi.c2) + static_cast<long long>(m0) * d.epi.ldc2 + (KIND == EPI_SWIGLU ? n0 / 2 : n0));
      constexpr int CM = KIND == EPI_DSWIGLU ? 4 : 2;       // bytes of c (and of h) per column of this contraction
      int rope_off[JP];                                     // rotation table: head row and pair of a lane's columns
      bool rope_on[JP];
      if constexpr (KIND == EPI_ROPE) {
#pragma unroll
        for (int jp = 0; jp < JP; ++jp) {
          const int n = nw + jp * 32, head = n / d.epi.rope_kp, row = head < d.epi.rope_hq ? head / d.epi.rope_qpk : head - d.epi.rope_hq;
          rope_on[jp] = n < d.epi.rope_cols;
          rope_off[jp] = rope_on[jp] ? (row * d.epi.rope_L) * (d.epi.rope_kp / 2) + (n % d.epi.rope_kp) / 2 : 0;
        }
      }
      // side inputs (saved pre-activations, rotation tables) of row block i: requested one block ahead of their use
      EpiSide nxt[JP];
      auto request = [&](int i) __attribute__((always_inline)) {
        const int row = min(row_l + i * 16, rows_in - 1);
        const int tpos = KIND == EPI_ROPE ? (m0 + row) % d.epi.rope_L * (d.epi.rope_kp / 2) : 0;
#pragma unroll
        for (int jp = 0; jp < JP; ++jp) {
          if constexpr (KIND == EPI_ROPE) {
            nxt[jp].a = *reinterpret_cast<const uint4*>(d.epi.rope_cos + rope_off[jp] + tpos);
            nxt[jp].b = *reinterpret_cast<const uint4*>(d.epi.rope_sin + rope_off[jp] + tpos);
          } else if constexpr (epi_has_side(KIND)) {
            const char* p = hb + static_cast<off_t>(row) * (static_cast<off_t>(d.epi.ldh) * 2u) + (cols_in ? nl + jp * 32 : min(nl + jp * 32, n_last)) * CM;
            nxt[jp].a = *reinterpret_cast<const uint4*>(p);
            if constexpr (KIND == EPI_DSWIGLU) nxt[jp].b = *reinterpret_cast<const uint4*>(p + 16);
          }
        }
      };
      if constexpr (epi_has_side(KIND)) request(0);
      auto side = [&](int i, EpiSide (&sd)[JP]) __attribute__((always_inline)) {
        if constexpr (epi_has_side(KIND)) {
#pragma unroll
          for (int jp = 0; jp < JP; ++jp) sd[jp] = nxt[jp];
          request(i + 1);            // behind the last block: its row is clamped, the values are not used
        }
      };
      auto store = [&](int row, const EpiOut (&out)[JP]) __attribute__((always_inline)) {
        const off_t off = static_cast<off_t>(row) * ldc2b + nl * CM;
        if (row < rows_in) {
#pragma unroll
          for (int jp = 0; jp < JP; ++jp) {
            if (cols_in || nl + jp * 32 <= n_last) {
              if (KIND != EPI_SWIGLU || d.epi.c) *reinterpret_cast<uint4*>(cb + off + jp * (32 * CM)) = out[jp].o[0];
              if constexpr (KIND == EPI_DSWIGLU) *reinterpret_cast<uint4*>(cb + off + jp * (32 * CM) + 16) = out[jp].o[1];
              if constexpr (KIND == EPI_BIAS_ACT)
                *reinterpret_cast<uint4*>(c2b + static_cast<off_t>(row) * (static_cast<off_t>(d.epi.ldc2) * 2u) + nl * 2 + jp * 64) = out[jp].a2;
              if constexpr (KIND == EPI_SWIGLU)
                *reinterpret_cast<uint2*>(c2b + static_cast<off_t>(row) * (static_cast<off_t>(d.epi.ldc2) * 2u) + nl + jp * 32) = make_uint2(out[jp].a2.x, out[jp].a2.y);
            }
          }
        }
      };
      constexpr bool GELU = KIND == EPI_BIAS_ACT || KIND == EPI_ACT || KIND == EPI_DACT;
      if constexpr (!PARK) {
        if (!GELU || !park) {
          ring_for<0, FM>([&](auto i_) __attribute__((always_inline)) {
            constexpr int i = decltype(i_)::value;
            EpiSide sd[JP];
            side(i, sd);
            EpiOut out[JP];
            ring_for<0, JP>([&](auto jp_) __attribute__((always_inline)) {
              constexpr int jp = decltype(jp_)::value;
              float v[8];
              vals(i_, jp_, v);
              add_bias(jp, v);
              epi_math_k<KIND>(ECOSPA_ACT_GELU_ERF, v, sd[jp], KIND == EPI_ROPE && rope_on[jp], out[jp]);
            });
            store(row_l + i * 16, out);
          });
          return;
        }
      }
      if constexpr (PARK || GELU) {
        ring_for<0, FM / CH>([&](auto ch_) __attribute__((always_inline)) {
          ring_for<0, CH>([&](auto i_) __attribute__((always_inline)) {
            ring_for<0, JP>([&](auto jp_) __attribute__((always_inline)) {
              float v[8];
              vals(ring_ic<decltype(ch_)::value * CH + decltype(i_)::value>{}, jp_, v);
              float4* s4 = reinterpret_cast<float4*>(slots + (decltype(i_)::value * JP + decltype(jp_)::value) * 2048);
              s4[0] = make_float4(v[0], v[1], v[2], v[3]);
              s4[64] = make_float4(v[4], v[5], v[6], v[7]);
            });
          });
#pragma unroll 1
          for (int il = 0; il < CH; ++il) {
            const int i = decltype(ch_)::value * CH + il;
            EpiSide sd[JP];
            side(i, sd);
            EpiOut out[JP];
#pragma unroll
            for (int jp = 0; jp < JP; ++jp) {
              const float4* s4 = reinterpret_cast<const float4*>(slots + (il * JP + jp) * 2048);
              const float4 lo = s4[0], hi = s4[64];
              float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
              add_bias(jp, v);
              epi_math_k<KIND>(PARK ? d.epi.act : ECOSPA_ACT_GELU_TANH, v, sd[jp], KIND == EPI_ROPE && rope_on[jp], out[jp]);
            }
            store(row_l + i * 16, out);
          }
        });
      }
    }
  });
}

template <int BM, int BN, int NS, bool TA, bool TB, bool CS, int EPIS, bool WIDE = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void gemm_bf16_ring_kernel(const RingGrid w, const GemmDesc d) {
  ring_tile<BM, BN, NS, TA, TB, CS, EPIS, WIDE>(d, w, blockIdx.x);
}

// ---------------------------------------------------------------------------------------------
// launch
template <int BM, int BN, int NS, bool TA, bool TB, bool CS, int EPIS, bool WIDE = false>
static hipError_t ring_launch_shape(ecospa_ctx* ctx, const GemmDesc& d, int k_chunk) {
  const int splits = d.splits > 1 ? d.splits : 1;
  const RingGrid w = gemm_ring_grid(d.M, d.N, BM, BN, splits, k_chunk);
  constexpr int lds_bytes = NS * (BM + BN) * RING_BK * static_cast<int>(sizeof(bf16_t));
  static_assert(lds_bytes <= 160 * 1024, "LDS of a compute unit");
  auto kern = gemm_bf16_ring_kernel<BM, BN, NS, TA, TB, CS, EPIS, WIDE>;
  static LdsAttrOnce attr_once;
  if (lds_bytes > 64 * 1024) {
    const hipError_t e = attr_once.ensure(reinterpret_cast<const void*>(kern), lds_bytes);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(w.tiles * splits), dim3(256), lds_bytes, ctx->stream, w, d);
  return hipGetLastError();
}

// Two contractions that do not depend on each other, a weight gradient dY^T X and an x W^T with a plain store, in one launch: the first
// n_tt workgroups take the tiles of the first.  Alone, each of the two pays for its launch (2.5 us), its first slabs (2 us) and its last
// stores with the matrix units idle, and often fills a part of the compute units only (when it is taken: pair_pays() in gemm.hip).
template <int TM, int TN, int TS, bool CS, int XM, int XN, int XS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void gemm_bf16_pair_kernel(const RingGrid wg, const RingGrid xg, int n_tt, const GemmDesc w, const GemmDesc x) {
  const int block = blockIdx.x;
  if (block < n_tt) ring_tile<TM, TN, TS, true, true, CS, GEMM_EPIS_TX, false>(w, wg, block);
  else ring_tile<XM, XN, XS, false, false, false, 1 << EPI_STORE, false>(x, xg, block - n_tt);
}
template <int TM, int TN, int TS, bool CS, int XM, int XN, int XS>
static hipError_t ring_launch_pair(ecospa_ctx* ctx, const GemmDesc& w, const GemmDesc& x, int w_k_chunk) {
  const int splits = w.splits > 1 ? w.splits : 1;
  const RingGrid wg = gemm_ring_grid(w.M, w.N, TM, TN, splits, w_k_chunk), xg = gemm_ring_grid(x.M, x.N, XM, XN, 1, (x.K + 63) / 64 * 64);
  const int n_tt = wg.tiles * splits;
  constexpr int lds_w = TS * (TM + TN) * RING_BK * 2, lds_x = XS * (XM + XN) * RING_BK * 2, lds_bytes = lds_w > lds_x ? lds_w : lds_x;
  static_assert(lds_bytes > 64 * 1024 && lds_bytes <= 160 * 1024, "LDS of a compute unit");
  auto kern = gemm_bf16_pair_kernel<TM, TN, TS, CS, XM, XN, XS>;
  static LdsAttrOnce attr_once;
  const hipError_t e = attr_once.ensure(reinterpret_cast<const void*>(kern), lds_bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(n_tt + xg.tiles), dim3(256), lds_bytes, ctx->stream, wg, xg, n_tt, w, x);
  return hipGetLastError();
}
