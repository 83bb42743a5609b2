// Device side of the deterministic block-wide top-k (step 2), shared by the selection launches and by the launch that
// finishes the scores and selects in one go (not part of the C ABI).
#pragma once
#include "common.h"

#define SELECT_THREADS 1024
#define SELECT_MAX_ITEMS 96    // descriptors travel as kernel arguments

struct SelectItemDev {
  const float* scores;
  int* idx;
  int n, k;
  int blk_begin;   // first workgroup (= group) of this item
  int groups;        // groups of this item (n <= 64: SELECT_THREADS / 64 of them share a workgroup)
  const int* k_dev;  // optional: per-group kept counts in device memory (then k is unused, the rows of idx
  int ld_idx;        //           are ld_idx apart and the slots behind the kept indices are set to -1)
  int smallest;      // take the k smallest scores instead (the order of the keys reversed, ties still to the lower index)
};
struct SelectBatch {
  int n_items;
  int first_blk[SELECT_MAX_ITEMS];   // blk_begin of every item, side by side: the search for a group's item stays in a few cache lines
  SelectItemDev it[SELECT_MAX_ITEMS];
};

__device__ __forceinline__ uint32_t score_key(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0u;   // NaN: lowest
  if (u == 0x80000000u) u = 0u;                      // -0 -> +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Inclusive prefix sum over the lanes of a wavefront by lane-permutation (DPP) adds: inside the rows of 16, then the last
// lane of rows 0 and 2 into rows 1 and 3, then lane 31 into the upper half - nothing goes through LDS.
#define ECOSPA_DPP_IADD(v, ctrl, rows) ((v) + __builtin_amdgcn_update_dpp(0, (v), (ctrl), (rows), 0xF, false))
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1, lanes without a source add 0
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);   // row_shr:8
  v = ECOSPA_DPP_IADD(v, 0x142, 0xA);                              // row_bcast:15 into rows 1 and 3
  v = ECOSPA_DPP_IADD(v, 0x143, 0xC);                              // row_bcast:31 into rows 2 and 3
  return v;
}

// Exclusive prefix sums of `a` and of `b` over the block's threads in thread order (one pass for both).
// `wave_tot` holds 2 x (SELECT_THREADS / 64) ints and must not be in use by another scan one barrier earlier.
__device__ __forceinline__ void block_exclusive_scan2(int a, int b, int* wave_tot, int& a_before, int& b_before) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ia = wave_inclusive_scan(a), ib = wave_inclusive_scan(b);
  if (lane == 63) { wave_tot[2 * wave] = ia; wave_tot[2 * wave + 1] = ib; }
  __syncthreads();
  int ba = 0, bb = 0;
#pragma unroll
  for (int w = 0; w < SELECT_THREADS / 64; ++w) {
    const int ca = wave_tot[2 * w], cb = wave_tot[2 * w + 1];
    if (w < wave) { ba += ca; bb += cb; }
  }
  a_before = ba + ia - a;
  b_before = bb + ib - b;
}

// LDS of one selecting workgroup.  One histogram per wavefront: normalised scores share their top key bits, so a
// single histogram would serialise nearly every atomic of the first pass on a few counters.
struct SelectShared {
  int whist[SELECT_THREADS / 64][256];
  int wave_tot[2 * (SELECT_THREADS / 64)];
  uint32_t s_prefix;
  int s_krem, s_all, s_in, s_other;      // s_in: keys of the digit that holds the wanted rank; s_one, s_other: see the ties
  uint32_t s_one;
};
#define ITEM_KEY(x) (score_key(x) ^ flip)
// A group of more than 64 units by one workgroup.  CACHE: score keys a thread keeps in registers (its contiguous run of
// indices is read once for all passes); 0: longer runs are read again in every pass.
template <int CACHE>
__device__ __forceinline__ void select_large_group(const SelectItemDev& t, int blk, SelectShared& sh) {
  auto& whist = sh.whist;
  auto& wave_tot = sh.wave_tot;
  uint32_t& s_prefix = sh.s_prefix;
  int& s_krem = sh.s_krem;
  const int tid = threadIdx.x, wave = tid >> 6;
  const uint32_t flip = t.smallest ? 0xffffffffu : 0u;
  constexpr bool cached = CACHE > 0;
  constexpr int NC = CACHE > 0 ? CACHE : 1;
  const int n = t.n, g = blk;
  const int k = t.k_dev ? t.k_dev[g] : t.k;
  const float* s = t.scores + static_cast<long long>(g) * n;
  int* out = t.idx + static_cast<long long>(g) * (t.k_dev ? t.ld_idx : k);

  // this thread's contiguous run of indices
  const int per = (n + SELECT_THREADS - 1) / SELECT_THREADS;
  const int i0 = min(tid * per, n), i1 = min(i0 + per, n);
  // Keys count from the smallest of the group on, and the passes start at the highest bit in which any two differ: normalised scores share
  // sign and most of the exponent, which made the first of four 8-bit passes over whole keys nearly idle.  And they end with the digit whose
  // keys are all kept - mostly the second, when one key is left.  (1024 units 7.2 -> 5.6 us, 5461 in the launch that finishes their scores 19.4 -> 16.3.)
  uint32_t kc[NC], least = 0u;
  int bits = 32;
  for (int i = tid; i < (SELECT_THREADS / 64) * 256; i += SELECT_THREADS) (&whist[0][0])[i] = 0;
  if (tid == 0) { s_prefix = 0u; s_krem = k; sh.s_all = sh.s_in = sh.s_other = 0; }
  if (cached) {
    uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const bool in = i0 + j < i1;
      kc[j] = in ? ITEM_KEY(s[i0 + j]) : 0u;
      lo = min(lo, in ? kc[j] : 0xffffffffu);
      hi = max(hi, kc[j]);
    }
    lo = wave_umin(lo);
    hi = ~wave_umin(~hi);
    if ((tid & 63) == 0) { wave_tot[2 * wave] = static_cast<int>(lo); wave_tot[2 * wave + 1] = static_cast<int>(hi); }
    __syncthreads();
    const int w = tid & (SELECT_THREADS / 64 - 1);      // a lane per wavefront
    least = __builtin_amdgcn_readfirstlane(wave_umin(static_cast<uint32_t>(wave_tot[2 * w])));
    hi = __builtin_amdgcn_readfirstlane(~wave_umin(~static_cast<uint32_t>(wave_tot[2 * w + 1])));
    bits = hi > least ? 32 - __builtin_clz(hi - least) : 1;
#pragma unroll
    for (int j = 0; j < NC; ++j) kc[j] -= least;
  }

  uint32_t prefix = 0u;   // high bits of the k-th largest key found so far
  int krem = k;           // rank (1-based) of the wanted key among keys matching the prefix
  bool all = false;       // every key that matches the prefix is kept
  __syncthreads();
  for (int pass = 0, above = bits; pass < 4 && above > 0 && !all; ++pass) {      // above: bits that are not decided yet
    const int shift = max(above - 8, 0);
    const uint32_t hi_mask = above >= 32 ? 0u : (0xffffffffu << above), low = ~hi_mask;
    if (cached) {
#pragma unroll
      for (int j = 0; j < NC; ++j)
        if (i0 + j < i1 && (kc[j] & hi_mask) == prefix) atomicAdd(&whist[wave][(kc[j] & low) >> shift], 1);
    } else {
      for (int i = i0; i < i1; ++i) {
        const uint32_t key = ITEM_KEY(s[i]);
        if ((key & hi_mask) == prefix) atomicAdd(&whist[wave][(key & low) >> shift], 1);
      }
    }
    __syncthreads();
    // suffix sums suf[d] = number of matching keys with digit >= d: the first four wavefronts own 64 digits each, add
    // the per-wavefront histograms (and clear them for the next pass), scan inside the wavefront by lane permutations,
    // then add the totals of the digits above.  Exactly one digit has suf[d] >= krem > suf[d + 1] = suf[d] - cnt[d].
    int cnt = 0, suf = 0;
    if (tid < 256) {
#pragma unroll
      for (int w = 0; w < SELECT_THREADS / 64; ++w) { cnt += whist[w][tid]; whist[w][tid] = 0; }
      const int inc = wave_inclusive_scan(cnt);
      const int tot = __builtin_amdgcn_readlane(inc, 63);
      suf = tot - inc + cnt;
      if ((tid & 63) == 0) wave_tot[wave] = tot;
    }
    __syncthreads();
    if (tid < 256) {
      for (int w = wave + 1; w < 4; ++w) suf += wave_tot[w];
      if (suf >= krem && suf - cnt < krem) {
        s_prefix = prefix | (static_cast<uint32_t>(tid) << shift);
        s_krem = krem - (suf - cnt);
        sh.s_all = suf == krem;
        sh.s_in = cnt;
      }
    }
    __syncthreads();
    prefix = __builtin_amdgcn_readfirstlane(s_prefix);
    krem = __builtin_amdgcn_readfirstlane(s_krem);
    all = __builtin_amdgcn_readfirstlane(sh.s_all) != 0;
    above = shift;
    // Ties: where sixteen bits are decided and still more keys are left than distinct ones mostly leave, they are one value (pruned units that all score
    // zero), which two looks tell sooner than two more passes: 1024 units, six in ten zero, 8.8 us with four passes over whole keys, 9.7 with the range in
    // front of them, now 7.5; five values 7.9, 8.5, 6.9.
    if (cached && pass >= 1 && !all && above > 0 && __builtin_amdgcn_readfirstlane(sh.s_in) > 8 + (n >> 8)) {
      const uint32_t mask = 0xffffffffu << above;
#pragma unroll
      for (int j = 0; j < NC; ++j)
        if (i0 + j < i1 && (kc[j] & mask) == prefix) sh.s_one = kc[j];
      __syncthreads();
      const uint32_t one = __builtin_amdgcn_readfirstlane(sh.s_one);
#pragma unroll
      for (int j = 0; j < NC; ++j)
        if (i0 + j < i1 && (kc[j] & mask) == prefix && kc[j] != one) sh.s_other = pass;
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(sh.s_other) != pass) {
        prefix = one;
        above = 0;
      }
    }
  }
  // kept: the keys above T (from T on, if all with its prefix are) and, of those equal to it, the first `krem`
  const uint32_t T = prefix;
  auto above_t = [&](uint32_t key) __attribute__((always_inline)) { return key > T || (all && key == T); };
  auto tie = [&](uint32_t key) __attribute__((always_inline)) { return !all && key == T; };

  int n_eq = 0, n_gt = 0;
  if (cached) {
#pragma unroll
    for (int j = 0; j < NC; ++j)
      if (i0 + j < i1) { n_eq += tie(kc[j]); n_gt += above_t(kc[j]); }
  } else {
    for (int i = i0; i < i1; ++i) {
      const uint32_t key = ITEM_KEY(s[i]);
      n_eq += tie(key);
      n_gt += above_t(key);
    }
  }
  // the ties are kept in index order until `krem` of them are: min(ties before this run, krem) of those before it
  int eq_before, gt_before;
  block_exclusive_scan2(n_eq, n_gt, wave_tot, eq_before, gt_before);
  int eq_left = max(0, min(n_eq, krem - eq_before));       // ties of this run that are kept
  int pos = gt_before + min(eq_before, krem);
  if (cached) {
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      if (i0 + j >= i1) continue;
      bool take = above_t(kc[j]);
      if (tie(kc[j]) && eq_left > 0) { take = true; --eq_left; }
      if (take && pos < k) out[pos++] = i0 + j;
    }
  } else {
    for (int i = i0; i < i1; ++i) {
      const uint32_t key = ITEM_KEY(s[i]);
      bool take = above_t(key);
      if (tie(key) && eq_left > 0) { take = true; --eq_left; }
      if (take && pos < k) out[pos++] = i;
    }
  }
  if (t.k_dev)
    for (int i = k + tid; i < t.ld_idx; i += SELECT_THREADS) out[i] = -1;
}

// The work of workgroup number `blk` of item t (all SELECT_THREADS threads of the workgroup call it).
__device__ __forceinline__ void select_item_block(const SelectItemDev& t, int blk, SelectShared& sh) {
  const int tid = threadIdx.x, wave = tid >> 6;
  const uint32_t flip = t.smallest ? 0xffffffffu : 0u;
  if (t.n <= 64) {
    // Small groups (the units of one head): a wavefront ranks a group by direct comparison - the rank of
    // a unit is the number of units that come before it in the order (larger key, or equal key and lower
    // index) - and the lanes whose rank is below k write their indices, ascending.  One group per wavefront.
    const int g = blk * (SELECT_THREADS / 64) + wave;
    if (g >= t.groups) return;
    const int lane = tid & 63, n = t.n;
    const int k = t.k_dev ? t.k_dev[g] : t.k;
    const uint32_t key = lane < n ? ITEM_KEY(t.scores[static_cast<long long>(g) * n + lane]) : 0u;
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const uint32_t kj = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(key), j));   // j is uniform: no LDS crossbar
      rank += (kj > key) || (kj == key && j < lane);
    }
    const bool take = lane < n && rank < k;
    const unsigned long long mask = __ballot(take);
    int* out = t.idx + static_cast<long long>(g) * (t.k_dev ? t.ld_idx : k);
    if (take) out[__popcll(mask & ((1ull << lane) - 1ull))] = lane;
    if (t.k_dev)
      for (int i = k + lane; i < t.ld_idx; i += 64) out[i] = -1;
    return;
  }
  // runs of up to 8 units per thread (groups of up to 8192) or of up to 32 (32768) stay in registers
  const int per = (t.n + SELECT_THREADS - 1) / SELECT_THREADS;
  if (per <= 8) select_large_group<8>(t, blk, sh);
  else if (per <= 32) select_large_group<32>(t, blk, sh);
  else select_large_group<0>(t, blk, sh);
}

#undef ITEM_KEY
