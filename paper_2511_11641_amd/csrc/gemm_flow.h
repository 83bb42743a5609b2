// The bf16 contraction kernel for launches of more tiles than compute units (not part of the C ABI).
//
// Main loop, LDS layout, fragments and products are those of gemm_ring.h.  What differs: 256 resident workgroups, one per compute unit,
// walk the output tiles, and nothing stops between two of them.
//   * The stream of operand slabs runs on over tile borders: while the last slabs of a tile are multiplied, the first ones of the next
//     tile are on their way into the ring.
//   * A finished tile's accumulators are copied aside (512 registers per lane hold both sets), and its epilogue - side inputs, activation,
//     conversion, stores - is dealt evenly over the matrix instructions of the next tile's first FLOW_NB slabs, one or two vector
//     instructions behind each.
// Why: in the kernel of one tile per workgroup everything but the main loop is exposed, once per round of tiles, 4.9 us with plain stores
// and 192x192 tiles (stores alone move 6.2 TB/s, so a round of bf16 tiles is 3 us of them; the first slabs take 2 us), more with an activation.  Here
// 2.3 us of a round remain.  The main loop is limited by power (a slab of 256x128 tiles takes 0.51 us on zeros, 0.70 us on N(0,1) operands),
// so its own instructions count twice: addresses and buffer numbers move between the products, the next tile is aimed at in one slab of its
// own, and the loop is as fast as the unrolled one (0.77 us per slab of 192x192).  Stores dealt over four slabs instead of twelve cost 0.7 us
// a slab: their acknowledgements come back in order with the loads that the ring waits for.
// 192x192 because it has the best rate of the tiles whose two accumulator sets fit.  N(0,1) operands, x W^T, 2048 tiles, kernel of one tile
// per workgroup -> this one: K = 1024 135 -> 119 us, 2048 229 -> 219, 4096 423 -> 417; in a layer's pass (operands and outputs cold):
// 4096x11008x2048 with SwiGLU 219 -> 170 us, 4096x6144x2048 with rotation 118 -> 104, dY^T X 4096x8256x2048 151 -> 123.
//
// Every store is issued whatever the tile's edge: rows and columns beyond the matrix repeat its last ones in the operand tiles, so their
// values are equal to those of the rows and columns they repeat and are written there once more.  That keeps the count of memory
// operations behind a slab's loads known (the waits name it).
#pragma once
#include "gemm_ring.h"

#define FLOW_BM GEMM_FLOW_TILE
#define FLOW_BN GEMM_FLOW_TILE
#define FLOW_NS 3
#define FLOW_NB 13
#define FLOW_MIN_SLABS GEMM_FLOW_MIN_SLABS

// Direct loads of one operand tile: as RingLoads, for whole slabs, re-aimed for every tile.
template <int RT, bool KSLOW>
struct FlowLoads {
  static constexpr int PER = RT * RING_BK * 2 / 1024 / 4;
  const char* base;
  unsigned off[PER];
  long long step;
  // EIGHTS: rows beyond the matrix repeat its last eight (the rows of a K-contiguous B, whose number is a multiple of eight), otherwise the last one
  template <bool EIGHTS>
  __device__ __forceinline__ void aim(const bf16_t* mat, long long ld, int r0, int R) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    base = reinterpret_cast<const char*>(KSLOW ? mat + r0 : mat + static_cast<long long>(r0) * ld);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int p = (wave * PER + i) * 64 + lane;
      int r, k;
      if constexpr (!KSLOW) {
        r = p / 8;
        k = ((p % 8) ^ (r & 7)) * 8;
      } else {
        k = p / (RT / 8);
        r = ((p % (RT / 8)) ^ ring_ks_swz<RT>(k)) * 8;
      }
      int gr;
      if constexpr (KSLOW) gr = min(r, R - 8 - r0);
      else if constexpr (EIGHTS) gr = r0 + r < R ? r : R - 8 - r0 + (r & 7);
      else gr = min(r, R - 1 - r0);
      const unsigned l = static_cast<unsigned>(ld), ur = static_cast<unsigned>(gr), uk = static_cast<unsigned>(k);
      off[i] = (KSLOW ? uk * l + ur : ur * l + uk) * 2u;
    }
    step = KSLOW ? static_cast<long long>(RING_BK) * ld * 2 : RING_BK * 2;
  }
  __device__ __forceinline__ void hold() { base -= step; step = 0; }      // no further tile: the last slab again and again
  __device__ __forceinline__ void issue(int i, lds_bf16_t* tile) {       // tile: where this wavefront's share of it begins
    asm volatile("" : "+v"(off[i]));
    __builtin_amdgcn_global_load_lds(reinterpret_cast<const void*>(base + off[i]), tile + i * 512, 16, 0, 0);
    if (i == PER - 1) base += step;
  }
};

// The epilogue of 8 consecutive columns of a row, cut into pieces of a few vector instructions: four that take the values out of the
// accumulators, two that add the bias, then the kind's own stages on four values at a time, and one that packs and stores.
template <int KIND>
struct FlowEpi {
  static constexpr int STAGES = KIND == EPI_BIAS_ACT || KIND == EPI_ACT ? 9 : KIND == EPI_DACT ? 10 : KIND == EPI_SWIGLU ? 3 : KIND == EPI_DSWIGLU ? 8 : KIND == EPI_ROPE ? 2 : 0;
  static constexpr bool BIAS = KIND != EPI_DACT && KIND != EPI_DSWIGLU;
  static constexpr int P0 = 4, P1 = P0 + (BIAS ? 2 : 0), PIECES = P1 + 2 * STAGES + 1;
  static constexpr int SIDES = KIND == EPI_DACT ? 1 : KIND == EPI_DSWIGLU || KIND == EPI_ROPE ? 2 : 0;      // side inputs per group: loads
  static constexpr int STORES = KIND == EPI_DSWIGLU || KIND == EPI_BIAS_ACT ? 2 : 1;                        // stores per group, at least
  float x[8], z[8], t[8], p[8], e[8], h[8];

  // stage ST of value q; sd: side inputs
  template <int ST>
  __device__ __forceinline__ void stage(int q, const EpiSide& sd, bool rope_on) {
    if constexpr (KIND == EPI_BIAS_ACT || KIND == EPI_ACT || KIND == EPI_DACT) {
      // act_norm_tail() of x (of the saved pre-activation for the derivative) and what follows from it, a step per stage
      if constexpr (KIND == EPI_DACT && ST == 0) {
        const uint32_t w[4] = {sd.a.x, sd.a.y, sd.a.z, sd.a.w};
        h[q] = __uint_as_float(q & 1 ? w[q >> 1] & 0xffff0000u : w[q >> 1] << 16);
      }
      const float a = KIND == EPI_DACT ? h[q] : x[q];
      if constexpr (ST == 0) t[q] = act_tail_t(a);
      if constexpr (ST == 1) p[q] = __builtin_fmaf(0.5307027145f, t[q], -0.7265760135f);
      if constexpr (ST == 2) p[q] = __builtin_fmaf(p[q], t[q], 0.7107068705f);
      if constexpr (ST == 3) p[q] = __builtin_fmaf(p[q], t[q], -0.142248368f);
      if constexpr (ST == 4) p[q] = __builtin_fmaf(p[q], t[q], 0.127414796f);
      if constexpr (ST == 5) e[q] = act_gauss(a);
      if constexpr (ST == 6) p[q] = p[q] * t[q];
      if constexpr (ST == 7) p[q] = p[q] * e[q];
      if constexpr (ST == 8) {
        if constexpr (KIND == EPI_DACT) z[q] = a < 0.f ? p[q] : 1.f - p[q];
        else z[q] = act_gelu_of_tail(a, p[q]);
      }
      if constexpr (ST == 9) x[q] *= __builtin_fmaf(a, 0.3989422804014327f * e[q], z[q]);
    } else if constexpr (KIND == EPI_SWIGLU) {
      // columns are (gate, up) pairs: four units, two steps per stage; e: denominator of the sigmoid, t: its reciprocal
      const int u = q & 3;
      if constexpr (ST == 0) {
        if (q < 4) e[u] = act_sigmoid_den(__expf(-x[2 * u]));
        else t[u] = __builtin_amdgcn_rcpf(e[u]);
      }
      if constexpr (ST == 1) {
        if (q < 4) t[u] = act_sigmoid_step(e[u], t[u]);
        else t[u] = act_sigmoid_end(e[u], t[u]);
      }
      if constexpr (ST == 2) {
        if (q < 4) z[u] = x[2 * u] * t[u];
        else z[u] = z[u] * x[2 * u + 1];
      }
    } else if constexpr (KIND == EPI_DSWIGLU) {
      const uint32_t w[8] = {sd.a.x, sd.a.y, sd.a.z, sd.a.w, sd.b.x, sd.b.y, sd.b.z, sd.b.w};
      const float g = __uint_as_float(w[q] << 16), u = __uint_as_float(w[q] & 0xffff0000u);
      if constexpr (ST == 0) e[q] = act_sigmoid_den(__expf(-g));
      if constexpr (ST == 1) t[q] = __builtin_amdgcn_rcpf(e[q]);
      if constexpr (ST == 2) t[q] = act_sigmoid_step(e[q], t[q]);
      if constexpr (ST == 3) t[q] = act_sigmoid_end(e[q], t[q]);
      if constexpr (ST == 4) z[q] = x[q] * u * t[q];
      if constexpr (ST == 5) p[q] = 1.f + g * (1.f - t[q]);
      if constexpr (ST == 6) z[q] *= p[q];
      if constexpr (ST == 7) p[q] = x[q] * g * t[q];
    } else if constexpr (KIND == EPI_ROPE) {
      const float4 c4 = __builtin_bit_cast(float4, sd.a), s4 = __builtin_bit_cast(float4, sd.b);
      const float cv[4] = {c4.x, c4.y, c4.z, c4.w}, sv[4] = {s4.x, s4.y, s4.z, s4.w};
      const int i = q >> 1;
      // which product is fused is written out: as in the wide tile shapes of the other kernel, so that the route does not decide the last bit
      if constexpr (ST == 0) z[q] = q & 1 ? __builtin_fmaf(x[q], cv[i], x[q - 1] * sv[i]) : __builtin_fmaf(x[q], cv[i], -(x[q + 1] * sv[i]));
      if constexpr (ST == 1) x[q] = rope_on ? z[q] : x[q];
    }
  }
};

// How the pieces of a tile's epilogue are dealt over the products of the next tile's first NB slabs: evenly over the products of slabs
// 1 .. NB - 1 (slab 0 only requests what the first ones read).
template <int BM, int BN, int KIND, int NB>
struct FlowDeal {
  static constexpr int FM = BM / 32, FN = BN / 32, NM = FM * FN, GROUPS = FM * FN / 2;
  static constexpr int SLOTS = (NB - 1) * 2 * NM, TOTAL = GROUPS * FlowEpi<KIND>::PIECES;
  static constexpr int first(int step, int m) { return step < 2 ? 0 : ((step - 2) * NM + m) * TOTAL / SLOTS; }        // first piece of product m of k step `step`
  static constexpr int groups_done(int step) { return first(step, 0) / FlowEpi<KIND>::PIECES; }                       // stored before that k step
  // groups whose side inputs have been requested before slab b: those that slab b + 1 begins with or reads
  static constexpr int requested(int b) { return b <= 0 ? 0 : (groups_upto(b + 2) < GROUPS ? groups_upto(b + 2) : GROUPS); }
  static constexpr int groups_upto(int b) { return 2 * b <= 2 ? 0 : b >= NB ? GROUPS : (first(2 * b, 0) + FlowEpi<KIND>::PIECES - 1) / FlowEpi<KIND>::PIECES; }
};

template <int BM, int BN, int NS, bool TA, bool TB, int KIND, int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void gemm_bf16_flow_kernel(const GemmDesc d, int tiles_n, int tiles) {
  constexpr int WTM = BM / 2, WTN = BN / 2, FM = WTM / 16, FN = WTN / 16, S = RING_BK / 32, NM = FM * FN, NR = FM + FN, JP = FN / 2;
  constexpr int STAGE = (BM + BN) * RING_BK;
  typedef FlowEpi<KIND> Epi;
  typedef FlowDeal<BM, BN, KIND, NB> Deal;
  constexpr int GROUPS = Deal::GROUPS;
  static_assert(S == 2 && FN % 2 == 0, "tile");
  extern __shared__ __attribute__((aligned(16))) bf16_t lds[];
  lds_bf16_t* lds3 = (lds_bf16_t*)lds;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = __builtin_amdgcn_readfirstlane(wave & 1), l16 = lane & 15, g = lane >> 4;

  // Every XCD owns a contiguous range of tiles (order as in gemm_ring.h), its workgroups take them in turn.
  constexpr int GROUP_M = BM >= 192 ? 4 : (BM >= 128 ? 8 : 16);
  const int tiles_m = tiles / tiles_n, xcd = blockIdx.x & 7, nwg = gridDim.x >> 3;
  const int per_xcd = tiles >> 3, more = tiles & 7;
  int id = xcd * per_xcd + min(xcd, more) + (blockIdx.x >> 3);
  const int id_end = xcd * per_xcd + min(xcd, more) + per_xcd + (xcd < more ? 1 : 0);
  auto place = [&](int t, int& m0, int& n0) __attribute__((always_inline)) {
    const int band = t / (GROUP_M * tiles_n), in_band = t - band * (GROUP_M * tiles_n);
    const int band_rows = min(GROUP_M, tiles_m - band * GROUP_M), col = in_band / band_rows;
    m0 = (band * GROUP_M + in_band - col * band_rows) * BM;
    n0 = col * BN;
  };
  const int nk = d.K / RING_BK;

  ring_f4 acc[FM][FN], park[FM][FN];
  FlowLoads<BM, TA> la;
  FlowLoads<BN, TB> lb;
  constexpr int PA = FlowLoads<BM, TA>::PER, PB = FlowLoads<BN, TB>::PER, LPW = PA + PB;
  int m0, n0;
  place(id, m0, n0);
  auto aim = [&](int am, int an) __attribute__((always_inline)) {
    la.template aim<false>(static_cast<const bf16_t*>(d.A), d.lda, am, d.M);
    lb.template aim<true>(static_cast<const bf16_t*>(d.B), d.ldb, an, d.N);
  };
  aim(m0, n0);
  const int swave = __builtin_amdgcn_readfirstlane(wave);
  lds_bf16_t* const lda0 = lds3 + swave * (PA * 512);
  lds_bf16_t* const ldb0 = lds3 + BM * RING_BK + swave * (PB * 512);
  int lbuf = 0;                 // buffer of the slab that is being loaded (elements)
  auto issue = [&](auto q_) __attribute__((always_inline)) {
    constexpr int q = decltype(q_)::value;
    if constexpr (q < PA) la.issue(q, lda0 + lbuf);
    else lb.issue(q - PA, ldb0 + lbuf);
  };
  auto next_buf = [&](int b) __attribute__((always_inline)) { return b == (NS - 1) * STAGE ? 0 : b + STAGE; };
  constexpr int LSTEPS = NS == 2 ? S - 1 : S;
  constexpr int LPS = (LPW + LSTEPS - 1) / LSTEPS;
  ring_for<0, NS - 1>([&](auto) __attribute__((always_inline)) {
    ring_for<0, LPW>([&](auto q_) __attribute__((always_inline)) { issue(q_); });
    lbuf = next_buf(lbuf);
  });
  RingFrags<BM, TA, FM> ra;
  RingFrags<BN, TB, FN> rb;
  ra.init(lds, wm * WTM);
  rb.init(lds + BM * RING_BK, wn * WTN);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(ring_waitcnt((NS - 2) * LPW, false));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  RingFrag fa[2][FM], fb[2][FN];
  // Addresses of the next fragment reads: K-contiguous one for each of the two k steps, moved to the next buffer while the reads of the
  // other step go out; K-slow one per fragment for both steps, moved behind the reads of step 1.
  constexpr int DA = TA ? FM : 1, DB = TB ? FN : 1;
  unsigned ada[TA ? 1 : 2][DA], adb[TB ? 1 : 2][DB];
  auto rd = [&](auto set_, auto s_, auto f_) __attribute__((always_inline)) {
    constexpr int set = decltype(set_)::value, s = decltype(s_)::value, f = decltype(f_)::value;
    constexpr bool isb = f >= 1 && f <= FN;
    constexpr int i = f == 0 ? 0 : (isb ? f - 1 : f - FN);
    constexpr bool ks = isb ? TB : TA;
    constexpr int RT = isb ? BN : BM;
    constexpr int imm = ks ? s * 32 * RT * 2 : i * 16 * RING_BK * 2;
    RingFrag& r = isb ? fb[set][i] : fa[set][i];
    const unsigned ad = isb ? adb[TB ? 0 : s][ks ? i : 0] : ada[TA ? 0 : s][ks ? i : 0];
    if constexpr (ks) {
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r.lo) : "v"(ad), "n"(imm));
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r.hi) : "v"(ad), "n"(imm + 4 * RT * 2));
    } else {
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r.v) : "v"(ad), "n"(imm));
    }
  };
  auto point = [&](auto s_, auto u_, int buf) __attribute__((always_inline)) {      // address u of step s into buffer buf (elements)
    constexpr int s = decltype(s_)::value, u = decltype(u_)::value;
    if constexpr (u < DA) ada[TA ? 0 : s][u] = ra.addr[TA ? u : s] + 2 * buf;
    else adb[TB ? 0 : s][u - DA] = rb.addr[TB ? u - DA : s] + 2 * buf;
  };
  auto landed = [&](auto set_) __attribute__((always_inline)) {
    constexpr int set = decltype(set_)::value;
    ring_for<0, FM>([&](auto i_) __attribute__((always_inline)) { ring_tie<TA>(fa[set][decltype(i_)::value]); });
    ring_for<0, FN>([&](auto j_) __attribute__((always_inline)) { ring_tie<TB>(fb[set][decltype(j_)::value]); });
    __builtin_amdgcn_sched_barrier(0);
  };
  int rbuf = 0;                 // buffer that is multiplied (elements)
  ring_for<0, DA + DB>([&](auto u_) __attribute__((always_inline)) {
    point(ring_ic<0>{}, u_, 0);
    point(ring_ic<1>{}, u_, 0);
  });
  ring_for<0, NR>([&](auto f_) __attribute__((always_inline)) { rd(ring_ic<0>{}, ring_ic<0>{}, f_); });
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  landed(ring_ic<0>{});

  // ---- epilogue of the parked tile --------------------------------------------------------------------------------------------------
  constexpr int CM = KIND == EPI_DSWIGLU ? 4 : 2;       // bytes of c (and of h) per column of this contraction
  Epi ep;
  EpiSide side[epi_has_side(KIND) ? GROUPS : 1];      // (a few of them live at a time)
  float bias[Epi::BIAS ? JP : 1][8];
  uint4 braw[JP];
  int pm0 = 0, pn0 = 0;
  int col[JP], rope_off[KIND == EPI_ROPE ? JP : 1];
  bool rope_on[KIND == EPI_ROPE ? JP : 1];
  const bool has_bias = Epi::BIAS && d.epi.bias != nullptr;
  const unsigned ldcb = static_cast<unsigned>(d.epi.ldc) * 2u, ldhb = static_cast<unsigned>(d.epi.ldh) * 2u, ldc2b = static_cast<unsigned>(d.epi.ldc2) * 2u;
  char *cb = nullptr, *c2b = nullptr;
  const char* hb = nullptr;
  auto row_of = [&](int i) __attribute__((always_inline)) {      // row of the tile whose values a lane holds in row block i
    const int r = wm * WTM + l16 + i * 16, in = d.M - pm0;
    if constexpr (TA) return r < in ? r : in - 8 + (r & 7);
    else return min(r, in - 1);
  };
  auto epi_aim = [&]() __attribute__((always_inline)) {          // the tile at pm0, pn0; requests its bias
    const int n_last = d.N - 8 - pn0, nl = wn * WTN + 16 * (g & 1) + 8 * (g >> 1);
    cb = reinterpret_cast<char*>(static_cast<bf16_t*>(d.epi.c) + static_cast<long long>(pm0) * d.epi.ldc + (KIND == EPI_DSWIGLU ? 2 * pn0 : pn0));
    if constexpr (KIND == EPI_BIAS_ACT || KIND == EPI_SWIGLU)
      c2b = reinterpret_cast<char*>(static_cast<bf16_t*>(d.epi.c2) + static_cast<long long>(pm0) * d.epi.ldc2 + (KIND == EPI_SWIGLU ? pn0 / 2 : pn0));
    if constexpr (KIND == EPI_DACT || KIND == EPI_DSWIGLU)
      hb = reinterpret_cast<const char*>(static_cast<const bf16_t*>(d.epi.h) + static_cast<long long>(pm0) * d.epi.ldh + (KIND == EPI_DSWIGLU ? 2 * pn0 : pn0));
#pragma unroll
    for (int jp = 0; jp < JP; ++jp) {
      col[jp] = min(nl + jp * 32, n_last);
      if constexpr (Epi::BIAS) braw[jp] = has_bias ? *reinterpret_cast<const uint4*>(static_cast<const bf16_t*>(d.epi.bias) + pn0 + col[jp]) : make_uint4(0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u);
      if constexpr (KIND == EPI_ROPE) {
        const int n = pn0 + col[jp], head = n / d.epi.rope_kp, row = head < d.epi.rope_hq ? head / d.epi.rope_qpk : head - d.epi.rope_hq;
        rope_on[jp] = n < d.epi.rope_cols;
        rope_off[jp] = rope_on[jp] ? (row * d.epi.rope_L) * (d.epi.rope_kp / 2) + (n % d.epi.rope_kp) / 2 : 0;
      }
    }
  };
  auto epi_bias = [&]() __attribute__((always_inline)) {
    if constexpr (Epi::BIAS) {
#pragma unroll
      for (int jp = 0; jp < JP; ++jp) unpack8(braw[jp], bias[jp]);
    }
  };
  auto request = [&](auto g_) __attribute__((always_inline)) {   // side inputs of group g
    constexpr int gi = decltype(g_)::value, i = gi / JP, jp = gi % JP;
    if constexpr (epi_has_side(KIND) && gi < GROUPS) {
      EpiSide& sd = side[gi];
      const int row = row_of(i);
      if constexpr (KIND == EPI_ROPE) {
        const int tpos = (pm0 + row) % d.epi.rope_L * (d.epi.rope_kp / 2);
        sd.a = *reinterpret_cast<const uint4*>(d.epi.rope_cos + rope_off[jp] + tpos);
        sd.b = *reinterpret_cast<const uint4*>(d.epi.rope_sin + rope_off[jp] + tpos);
      } else {
        const char* p = hb + static_cast<unsigned>(row) * ldhb + col[jp] * CM;
        sd.a = *reinterpret_cast<const uint4*>(p);
        if constexpr (KIND == EPI_DSWIGLU) sd.b = *reinterpret_cast<const uint4*>(p + 16);
      }
    }
  };
  auto piece = [&](auto g_, auto p_, ring_f4 (&from)[FM][FN]) __attribute__((always_inline)) {
    constexpr int gi = decltype(g_)::value, p = decltype(p_)::value, i = gi / JP, jp = gi % JP;
    if constexpr (gi < GROUPS) {
      const EpiSide& sd = side[epi_has_side(KIND) ? gi : 0];
      if constexpr (p < Epi::P0) {
        const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(from[i][2 * jp][p]), __float_as_uint(from[i][2 * jp + 1][p]), false, false);
        ep.x[p] = __uint_as_float(w[0]);
        ep.x[4 + p] = __uint_as_float(w[1]);
      } else if constexpr (p < Epi::P1) {
#pragma unroll
        for (int q = 4 * (p - Epi::P0); q < 4 * (p - Epi::P0) + 4; ++q) ep.x[q] += bias[Epi::BIAS ? jp : 0][q];
      } else if constexpr (p < Epi::PIECES - 1) {
        constexpr int st = (p - Epi::P1) / 2, q0 = 4 * ((p - Epi::P1) % 2);
#pragma unroll
        for (int q = q0; q < q0 + 4; ++q) ep.template stage<st>(q, sd, rope_on[KIND == EPI_ROPE ? jp : 0]);
      } else {
        const int row = row_of(i);
        char* const c = cb + (static_cast<unsigned>(row) * ldcb + static_cast<unsigned>(col[jp] * CM));
        if constexpr (KIND == EPI_DSWIGLU) {
          float o[2][8];
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            o[q >> 2][2 * (q & 3)] = ep.z[q];
            o[q >> 2][2 * (q & 3) + 1] = ep.p[q];
          }
          *reinterpret_cast<uint4*>(c) = pack8(o[0]);
          *reinterpret_cast<uint4*>(c + 16) = pack8(o[1]);
        } else if constexpr (KIND == EPI_ACT) {
          *reinterpret_cast<uint4*>(c) = pack8(ep.z);
        } else {
          if (KIND != EPI_SWIGLU || d.epi.c) *reinterpret_cast<uint4*>(c) = pack8(ep.x);
          if constexpr (KIND == EPI_BIAS_ACT)
            *reinterpret_cast<uint4*>(c2b + (static_cast<unsigned>(row) * ldc2b + static_cast<unsigned>(col[jp] * 2))) = pack8(ep.z);
          if constexpr (KIND == EPI_SWIGLU) {
            const uint4 a = pack8(ep.z);
            *reinterpret_cast<uint2*>(c2b + (static_cast<unsigned>(row) * ldc2b + static_cast<unsigned>(col[jp]))) = make_uint2(a.x, a.y);
          }
        }
      }
    }
  };

  constexpr int RSLOTS = NM * 3 / 4;        // as in gemm_ring.h
  // One slab.  EB: number of the slab in its tile while it carries a share of the parked tile's epilogue, -1 without; ZERO: the
  // accumulators start from zero; AIM: the loads reach the end of their tile.
  auto slab = [&](auto eb_, auto zero_, auto aim_) __attribute__((always_inline)) {
    constexpr int EB = decltype(eb_)::value;
    constexpr bool ZERO = decltype(zero_)::value != 0, AIM = decltype(aim_)::value != 0;
    ring_for<0, S>([&](auto s_) __attribute__((always_inline)) {
      constexpr int s = decltype(s_)::value;
      constexpr int cur = s & 1, nxt = cur ^ 1;
      constexpr bool last = s + 1 == S;
      constexpr int ls = last ? 0 : s + 1;
      constexpr int Q0 = ls * LPS < LPW ? ls * LPS : LPW, Q1 = (ls + 1) * LPS < LPW ? (ls + 1) * LPS : LPW, NQ = Q1 - Q0;
      if constexpr (AIM && last) {
        if (id + nwg < id_end) {
          int am, an;
          place(id + nwg, am, an);
          aim(am, an);
        } else {
          la.hold();
          lb.hold();
        }
      }
      if constexpr (EB == 0 && s == 0) epi_aim();
      if constexpr (EB == 1 && s == 0) epi_bias();
      if constexpr (EB >= 0 && s == 0 && epi_has_side(KIND))
        ring_for<Deal::requested(EB), Deal::requested(EB + 1)>([&](auto q_) __attribute__((always_inline)) { request(q_); });
      const int nbuf = next_buf(rbuf);
      __builtin_amdgcn_sched_barrier(0);
      ring_for<0, NM>([&](auto m_) __attribute__((always_inline)) {
        constexpr int m = decltype(m_)::value, i = m / FN, j = m % FN;
        const bf16x8_t b = ring_val<TB>(fb[cur][j]), a = ring_val<TA>(fa[cur][i]);
        if constexpr (ZERO && s == 0) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc[i][j]) : "v"(b), "v"(a));
        else ring_mfma(acc[i][j], b, a);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int R0 = m < RSLOTS ? m * NR / RSLOTS : NR, R1 = m < RSLOTS ? (m + 1) * NR / RSLOTS : NR;
        ring_for<R0, R1>([&](auto f_) __attribute__((always_inline)) { rd(ring_ic<nxt>{}, ring_ic<nxt>{}, f_); });
        ring_for<Q0 + m * NQ / NM, Q0 + (m + 1) * NQ / NM>([&](auto q_) __attribute__((always_inline)) { issue(q_); });
        // fragment addresses in the next slab's buffer
        constexpr int MV0 = RSLOTS + (last ? 1 : 0), U0 = m < MV0 ? 0 : (m - MV0) * (DA + DB) / (NM - MV0), U1 = m < MV0 ? 0 : (m + 1 - MV0) * (DA + DB) / (NM - MV0);
        ring_for<U0, U1>([&](auto u_) __attribute__((always_inline)) {
          constexpr bool ks = decltype(u_)::value < DA ? TA : TB;
          if constexpr (!ks || !last) point(s_, u_, nbuf);
        });
        if constexpr (EB >= 1)
          ring_for<Deal::first(2 * EB + s, m), Deal::first(2 * EB + s, m + 1)>([&](auto u_) __attribute__((always_inline)) {
            constexpr int u = decltype(u_)::value;
            piece(ring_ic<u / Epi::PIECES>{}, ring_ic<u % Epi::PIECES>{}, park);
          });
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr ((LSTEPS == 1) == last) lbuf = next_buf(lbuf);
      if constexpr (!last) {
        // Own loads of the next slab have landed.  Behind them are the loads of NS - 2 slabs and, at least, the stores of the last two
        // k steps and the side inputs requested in this one.
        constexpr int BEHIND = NS == 2 || EB < 0 ? 0 : (Deal::groups_done(2 * EB + 1) - Deal::groups_done(2 * EB - 1)) * Epi::STORES +
                                                       (epi_has_side(KIND) ? (Deal::requested(EB + 1) - Deal::requested(EB)) * Epi::SIDES : 0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(ring_waitcnt((NS - 2) * LPW + BEHIND, true));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      } else {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        rbuf = nbuf;
      }
      landed(ring_ic<nxt>{});
    });
  };
  ring_for<0, (LPS < LPW ? LPS : LPW)>([&](auto q_) __attribute__((always_inline)) { issue(q_); });
  if (LSTEPS == 1) lbuf = next_buf(lbuf);

  bool parked = false;
  for (;;) {
    int t;
    if (parked) {
      slab(ring_ic<0>{}, ring_ic<1>{}, ring_ic<0>{});
      ring_for<1, NB>([&](auto b_) __attribute__((always_inline)) { slab(b_, ring_ic<0>{}, ring_ic<0>{}); });
      t = NB;
    } else {
      slab(ring_ic<-1>{}, ring_ic<1>{}, ring_ic<0>{});
      t = 1;
    }
    for (; t < nk - NS; ++t) slab(ring_ic<-1>{}, ring_ic<0>{}, ring_ic<0>{});
    slab(ring_ic<-1>{}, ring_ic<0>{}, ring_ic<1>{});
    for (t = 1; t < NS; ++t) slab(ring_ic<-1>{}, ring_ic<0>{}, ring_ic<0>{});
    pm0 = m0;
    pn0 = n0;
    id += nwg;
    // the last products are still on their way into their accumulators
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) asm volatile("" : "+a"(acc[i][j]));
    __builtin_amdgcn_sched_barrier(0);
    if (id >= id_end) break;
    place(id, m0, n0);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) park[i][j] = acc[i][j];
    parked = true;
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 1" ::: "memory");
  }
  // the last tile has nothing to hide behind
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the repeated loads are still on their way into LDS
  epi_aim();
  epi_bias();
  ring_for<0, GROUPS>([&](auto g_) __attribute__((always_inline)) {
    if constexpr (decltype(g_)::value == 0) ring_for<0, 4>([&](auto q_) __attribute__((always_inline)) { request(q_); });
    request(ring_ic<decltype(g_)::value + 4>{});
    ring_for<0, Epi::PIECES>([&](auto p_) __attribute__((always_inline)) { piece(g_, p_, acc); });
  });
}

// ---------------------------------------------------------------------------------------------
// launch of a descriptor that gemm_flow_takes()
template <bool TA, bool TB, int KIND>
static hipError_t flow_launch(ecospa_ctx* ctx, const GemmDesc& d) {
  const int tm = (d.M + FLOW_BM - 1) / FLOW_BM, tn = (d.N + FLOW_BN - 1) / FLOW_BN;
  constexpr int lds_bytes = FLOW_NS * (FLOW_BM + FLOW_BN) * RING_BK * static_cast<int>(sizeof(bf16_t));
  static_assert(lds_bytes > 64 * 1024 && lds_bytes <= 160 * 1024, "LDS of a compute unit");
  static_assert(FLOW_MIN_SLABS >= FLOW_NB + FLOW_NS, "the loads turn to the next tile behind the epilogue");
  auto kern = gemm_bf16_flow_kernel<FLOW_BM, FLOW_BN, FLOW_NS, TA, TB, KIND, FLOW_NB>;
  static LdsAttrOnce attr_once;
  const hipError_t e = attr_once.ensure(reinterpret_cast<const void*>(kern), lds_bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(256), dim3(256), lds_bytes, ctx->stream, d, tn, tm * tn);
  return hipGetLastError();
}
