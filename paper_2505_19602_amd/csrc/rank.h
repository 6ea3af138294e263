// Ranking of one unit's cache by one workgroup (Eq. 5 and the top-k of Sec. 3.3, bf16): logits, row
// normalisers, log-scores, selection, index list.  rank_short: up to kShortLen rows, logits in LDS;
// rank_long: logits in registers, beyond them in the workspace.
//
// For short caches nothing is bound by bandwidth; the time is a chain of memory latencies and
// barriers.  The logits do not leave the compute unit (80 bytes of LDS a key: 16 window rows and a
// pad against bank conflicts), every wave forms the row normalisers itself instead of waiting for
// them, and the radix search skips the bits that all keys share and those that no longer matter:
// the first digit starts at the highest bit in which the largest and the smallest key differ, and
// the search ends as soon as the digit's bin is wanted whole.
//
// Every form selects the same rows bit for bit: groups of 32 keys belong to virtual waves group %
// 16, whose running maximum and sum are merged in group order, then in wave order.
#pragma once
#include "common.h"
#include "radix_select.h"
#include "score_mfma.h"

namespace scalekv {

constexpr int kShortGroups = kShortLen / 32;
constexpr int kLogitStride = 20;            // floats between the logits of consecutive keys in LDS
constexpr int kVirtualWaves = 16;           // waves of the general ranking kernel

struct RankShortLds {
  __attribute__((aligned(16))) uint32_t hist[4 * 256];
  float group_max[kShortGroups][kMaxWindow], group_sum[kShortGroups][kMaxWindow];
  uint32_t keys[kShortLen];
  int32_t list[kShortLen];                  // the selected rows, ascending
  uint32_t wave_max[16], wave_min[16];
  uint32_t count[kShortLen / 32];           // forced rows, a bit each; later per 64 keys how many are above and at the threshold
};
// dynamic LDS for the logits
inline int rank_short_logit_bytes(int len) { return round_up(len, 32) * kLogitStride * 4; }

// Maximum m and sum e of exponentials (above the maximum) of a window row over some keys, joined with those of others.  Every
// form joins by this function, and its roundings are written out: with them left to the compiler, forms that select the
// same rows today need not tomorrow.
__device__ __forceinline__ void join_keys(float& m, float& e, float m_more, float e_more) {
#pragma clang fp contract(off)
  const float top = fmaxf(m, m_more);
  e = fmaf(e, expf(m - top), e_more * expf(m_more - top));
  m = top;
}

// Rows in ascending order: thread tid holds the keys kk[c] of rows tid + c THREADS < len.  Those above T,
// the first need_eq equal to T and those whose bit c of `forced` is set go to list[] (LDS) and idx[], each
// if it is not NULL.  count: one word of LDS per 64 rows.  One barrier; the caller's next one publishes the list.
template <int THREADS, int PER>
__device__ __forceinline__ void emit_selected(const uint32_t (&kk)[PER], uint32_t forced, int len, uint32_t T,
                                              uint32_t need_eq, uint32_t* count, int32_t* list, int32_t* idx) {
  constexpr int kWaves = THREADS / 64;
  constexpr int PER_LANE = (PER * kWaves + 63) / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_slot = (len + 63) / 64;
  auto above = [&](int c) { return tid + c * THREADS < len && (kk[c] > T || (forced >> c & 1u)); };
  auto equal = [&](int c) { return tid + c * THREADS < len && kk[c] == T && !(forced >> c & 1u); };
#pragma unroll
  for (int c = 0; c < PER; ++c) {
    const int slot = c * kWaves + wave;
    if (slot < n_slot) {
      const uint32_t gt = __builtin_popcountll(__builtin_amdgcn_ballot_w64(above(c)));
      const uint32_t eq = __builtin_popcountll(__builtin_amdgcn_ballot_w64(equal(c)));
      if (lane == 0) count[slot] = gt | eq << 16;  // (both sums stay below 2^16)
    }
  }
  __syncthreads();
  uint32_t before[PER_LANE], carry = 0;
#pragma unroll
  for (int x = 0; x < PER_LANE; ++x) {
    const uint32_t mine = 64 * x + lane < n_slot ? count[64 * x + lane] : 0u;
    const uint32_t upto = wave_prefix_sum(mine, lane);
    before[x] = carry + upto - mine;
    carry += __builtin_amdgcn_readlane(upto, 63);
  }
#pragma unroll
  for (int c = 0; c < PER; ++c) {
    const int slot = c * kWaves + wave;
    if (slot < n_slot) {
      uint32_t base = 0;
#pragma unroll
      for (int x = 0; x < PER_LANE; ++x)
        if (slot / 64 == x) base = __builtin_amdgcn_readlane(before[x], slot % 64);
      const int key = tid + c * THREADS;
      const unsigned long long gt = __builtin_amdgcn_ballot_w64(above(c));
      const unsigned long long eq = __builtin_amdgcn_ballot_w64(equal(c));
      const unsigned long long below = ((unsigned long long)1 << lane) - 1;
      const uint32_t g_before = (base & 0xffffu) + __builtin_popcountll(gt & below);
      const uint32_t e_before = (base >> 16) + __builtin_popcountll(eq & below);
      const bool take = (gt >> lane & 1) || ((eq >> lane & 1) && e_before < need_eq);
      if (take) {
        const uint32_t pos = g_before + min(e_before, need_eq);
        if (list) list[pos] = key;
        if (idx) idx[pos] = key;
      }
    }
  }
}

// Largest and smallest of a value per thread, over the workgroup.  wave_max, wave_min: a word per wave.
template <int THREADS>
__device__ __forceinline__ void block_extremes(uint32_t& hi, uint32_t& lo, uint32_t* wave_max, uint32_t* wave_min) {
#define SCALEKV_ROW_ROR(v, n) (uint32_t) __builtin_amdgcn_update_dpp(0, (int)(v), 0x120 + (n), 0xf, 0xf, true)
  hi = max(hi, SCALEKV_ROW_ROR(hi, 8)), lo = min(lo, SCALEKV_ROW_ROR(lo, 8));
  hi = max(hi, SCALEKV_ROW_ROR(hi, 4)), lo = min(lo, SCALEKV_ROW_ROR(lo, 4));
  hi = max(hi, SCALEKV_ROW_ROR(hi, 2)), lo = min(lo, SCALEKV_ROW_ROR(lo, 2));
  hi = max(hi, SCALEKV_ROW_ROR(hi, 1)), lo = min(lo, SCALEKV_ROW_ROR(lo, 1));
#undef SCALEKV_ROW_ROR
  auto across = [](uint32_t x, auto join) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    const uint32_t y = join(r[0], r[1]);
    const auto s = __builtin_amdgcn_permlane32_swap(y, y, false, false);
    return join(s[0], s[1]);
  };
  hi = across(hi, [](uint32_t a, uint32_t b) { return max(a, b); });
  lo = across(lo, [](uint32_t a, uint32_t b) { return min(a, b); });
  if ((threadIdx.x & 63) == 0) { wave_max[threadIdx.x >> 6] = hi; wave_min[threadIdx.x >> 6] = lo; }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) {
    hi = max(hi, wave_max[w]);
    lo = min(lo, wave_min[w]);
  }
}

// Row normaliser max + log Z of window row i in every lane (g, i), by one wave: the lane brings maximum (-inf: no
// key) and sum of virtual waves 4g .. 4g+3 of that row.  Those of g >= turns are empty.  FUSED: the products of all
// turns are added unrounded, otherwise those of the first (the border of a selection may lie between scores that differ
// in the last bit: which rows are kept depends on every rounding here).
template <bool FUSED>
__device__ __forceinline__ float row_shift(const float (&vm)[4], const float (&ve)[4], int turns) {
#pragma clang fp contract(off)
  float mm = xor32_max(xor16_max(fmaxf(fmaxf(vm[0], vm[1]), fmaxf(vm[2], vm[3]))));
  float f[4];
#pragma unroll
  for (int x = 0; x < 4; ++x) f[x] = expf(vm[x] - mm);
  // the sum runs over the virtual waves in order: g = 0 hands its part to g = 1 and so on
  auto add = [&](float z, bool fused) __attribute__((always_inline)) {
#pragma clang fp contract(off)
#pragma unroll
    for (int x = 0; x < 4; ++x) z = !(vm[x] > -INFINITY) ? z : fused ? fmaf(ve[x], f[x], z) : z + ve[x] * f[x];
    return z;
  };
  float z = from_row<0>(add(0.f, true));
  if (turns > 1) z = from_row<1>(add(z, FUSED));
  if (turns > 2) z = from_row<2>(add(z, FUSED));
  if (turns > 3) z = from_row<3>(add(z, FUSED));
  return mm + logf(z);
}
// The same of all sixteen rows, as scalars.
__device__ __forceinline__ void row_shifts(float own, float (&shift)[kMaxWindow]) {
#pragma unroll
  for (int j = 0; j < kMaxWindow; ++j)
    shift[j] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(own), j));
}

// log_sum_rows (common.h) of one key by PARTS neighbouring lanes, each with 16 / PARTS of its window rows: `logits` are
// those of the key, `shift` is row_shift() of lane (g, i).  The terms are added in the order of the rows, the lanes in
// turn, so that every PARTS gives the same result.  A chain of 16 exponentials by a few of the waves is what a lane to a
// key costs; with it and the normalisers' chains shortened (row_shift, block_extremes in registers, logits stored
// without conditions) a step of 16 queries over 69 rows, 16 units, went from 9.8 to 9.2 us, 6 x 6 queries over 56 rows,
// 80 units, 9.3 to 8.9, ten maps of one image, 16 units, 172.6 to 168.1.
template <int PARTS>
__device__ __forceinline__ float log_sum_parts(const float* logits, int n_win, float shift) {
  static_assert(PARTS == 2 || PARTS == 4, "lanes of a row of four");
  constexpr int kOwn = kMaxWindow / PARTS;
  const int j0 = threadIdx.x % PARTS * kOwn;
  float la[kOwn], top = -INFINITY;
#pragma unroll
  for (int j = 0; j < kOwn; j += 4) {
    const float4 x = *(const float4*)(logits + j0 + j);
    la[j] = x.x; la[j + 1] = x.y; la[j + 2] = x.z; la[j + 3] = x.w;
  }
#pragma unroll
  for (int j = 0; j < kOwn; ++j) {
    const float row = __shfl(shift, j0 + j);
    la[j] = j0 + j < n_win ? la[j] - row : -INFINITY;
    top = fmaxf(top, la[j]);
  }
#define SCALEKV_QUAD(v, ctrl) \
  __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, true))
  top = fmaxf(top, SCALEKV_QUAD(top, 0xb1));                  // lane ^ 1
  if (PARTS == 4) top = fmaxf(top, SCALEKV_QUAD(top, 0x4e));  // lane ^ 2
#pragma unroll
  for (int j = 0; j < kOwn; ++j) la[j] = j0 + j < n_win ? expf(la[j] - top) : 0.f;
  auto add = [&](float z) {
#pragma unroll
    for (int j = 0; j < kOwn; ++j) z += la[j];
    return z;
  };
  // after turn t lane t of the key holds the sum so far; the others take it from there
  float z = add(0.f);
  if constexpr (PARTS == 4) {
    z = add(SCALEKV_QUAD(z, 0x00));
    z = add(SCALEKV_QUAD(z, 0x55));
    z = add(SCALEKV_QUAD(z, 0xaa));
    z = SCALEKV_QUAD(z, 0xff);
  } else {
    z = add(SCALEKV_QUAD(z, 0xa0));  // lanes 0 and 2
    z = SCALEKV_QUAD(z, 0xf5);       // lanes 1 and 3
  }
#undef SCALEKV_QUAD
  return top + logf(z);
}

// From the log-scores to the selection.  own[c]: log-score of row tid + c THREADS.  `keys` (LDS, len words)
// may hold other data until the first barrier if nothing is pooled; hist has been cleared.
template <int THREADS, int PER, bool EXTRAS, typename Lds>
__device__ __forceinline__ void select_scores(float (&own)[PER], int len, int keep, const SelectExtras& ex, Lds& lds,
                                              int32_t* list, int32_t* idx) {
  const int tid = threadIdx.x;
  if constexpr (EXTRAS) {
    if (ex.n_forced > 0) {  // (a bit per row: the list checked for every row costs 6 us at 12 rows a thread)
      static_assert(PER * THREADS <= 32 * THREADS, "a thread forms at most one word");
      if (tid < (len + 31) / 32) {
        uint32_t word = 0;
#pragma unroll  // (the list arrives with one scalar load; walked in a loop it costs 16 latencies)
        for (int j = 0; j < kMaxWindow; ++j)
          if (j < ex.n_forced && ex.forced[j] >> 5 == tid) word |= 1u << (ex.forced[j] & 31);
        lds.count[tid] = word;
      }
      __syncthreads();
    }
    if (ex.pool_w > 1) {
      float* raw = reinterpret_cast<float*>(lds.keys);
#pragma unroll
      for (int c = 0; c < PER; ++c)
        if (tid + c * THREADS < len) raw[tid + c * THREADS] = own[c];
      __syncthreads();
#pragma unroll
      for (int c = 0; c < PER; ++c)
        if (tid + c * THREADS < len)
          own[c] = pooled_log([&](int t) { return raw[t]; }, tid + c * THREADS, len, (ex.pool_w - 1) / 2);
      __syncthreads();
    }
  }
  // Forced rows take no part in the search (a key above all others for them would make the search start
  // at the sign bit, with all real keys in one bin: 512 units x 12000 close scores 62.1 us, 26.1 this way):
  // `keep` less their number is wanted of the others.
  uint32_t kk[PER];
  uint32_t hi = 0, lo = 0xffffffffu, forced = 0;
  int wanted = keep;
#pragma unroll
  for (int c = 0; c < PER; ++c) {
    const int key = tid + c * THREADS;
    kk[c] = 0;
    if (key < len) {
      kk[c] = order_key(own[c]);
      lds.keys[key] = kk[c];
      if constexpr (EXTRAS) {
        if (ex.n_forced > 0) forced |= (lds.count[key >> 5] >> (key & 31) & 1u) << c;
      }
      if (!(forced >> c & 1u)) {
        hi = max(hi, kk[c]);
        lo = min(lo, kk[c]);
      }
    }
  }
  if constexpr (EXTRAS) wanted -= ex.n_forced;
  block_extremes<THREADS>(hi, lo, lds.wave_max, lds.wave_min);
  // keys above T are selected, and the first need_eq of those equal to it
  uint32_t T = 0xffffffffu, need_eq = 0;
  if (!EXTRAS || wanted > 0)
    radix_kth_largest_from<THREADS, EXTRAS>([&](int t) { return lds.keys[t]; }, forced, len, (uint32_t)wanted,
                                            32 - __builtin_clz((hi ^ lo) | 1u), hi, lds.hist, T, need_eq);
  emit_selected<THREADS, PER>(kk, forced, len, T, need_eq, lds.count, list, idx);
  __syncthreads();
}

// The same for a few rows (len PARTS <= THREADS; own: log-score of row tid / PARTS) by counting, for every row, those with a
// larger score: PARTS lanes share a row, and each compares its key with a part of the others.  The radix search takes
// three or four barriers and as many round trips through LDS counters; this takes two.  False, with nothing
// emitted, if equal scores straddle the border: then it takes the search to choose among them.
// Whole steps, us, search / counting: 16 units, 16 queries, 69 rows 11.0 / 9.9; 128 rows 12.1 / 10.8; 200 rows (two parts)
// 12.7 / 12.3; head_dim 64, 69 rows 9.2 / 8.0; 256 units, 69 rows 12.9 / 11.4; 64 queries, 250 rows 21.7 / 21.5.
constexpr int kCountedRows = 256;  // longest for two parts: 128 comparisons a lane
template <int THREADS, int PARTS, typename Lds>
__device__ __forceinline__ bool select_by_rank(float own, int len, int keep, Lds& lds, int32_t* list, int32_t* idx) {
  constexpr int kWaves = THREADS / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int share = (len + 4 * PARTS - 1) / (4 * PARTS) * 4;  // keys per lane; a key of 0 beyond len is larger than none
  const int row = tid / PARTS;
  const uint32_t mine = row < len ? order_key(own) : 0u;
  if (tid % PARTS == 0 && row < share * PARTS) lds.keys[row] = mine;
  __syncthreads();
  const uint4* part = reinterpret_cast<const uint4*>(lds.keys + tid % PARTS * share);
  int above = 0;
#pragma unroll 4
  for (int j = 0; j < share / 4; ++j) {
    const uint4 x = part[j];
    above += (x.x > mine) + (x.y > mine) + (x.z > mine) + (x.w > mine);
  }
  above += __builtin_amdgcn_update_dpp(0, above, 0xb1, 0xf, 0xf, true);             // lane ^ 1
  if (PARTS == 4) above += __builtin_amdgcn_update_dpp(0, above, 0x4e, 0xf, 0xf, true);  // lane ^ 2
  const bool take = row < len && above < keep;
  const unsigned long long taken = __builtin_amdgcn_ballot_w64(take && tid % PARTS == 0);
  if (lane == 0) lds.count[wave] = __builtin_popcountll(taken);
  __syncthreads();
  const uint32_t counted = lane < kWaves ? lds.count[lane] : 0u;
  const uint32_t upto = wave_prefix_sum(counted, lane);
  if (__builtin_amdgcn_readlane(upto, 63) != (uint32_t)keep) return false;
  const uint32_t before = wave > 0 ? __builtin_amdgcn_readlane(upto, wave - 1) : 0u;
  if (taken >> lane & 1) {
    const uint32_t pos = before + __builtin_popcountll(taken & (((unsigned long long)1 << lane) - 1));
    list[pos] = row;
    if (idx) idx[pos] = row;
  }
  __syncthreads();
  return true;
}

// Leaves the `keep` selected rows in lds.list (0 < keep < len <= kShortLen) and, if idx is not
// NULL, in idx.  All THREADS threads of the workgroup call it; `logits` may be overwritten
// afterwards without a barrier.
template <int D, int THREADS, bool EXTRAS>
__device__ __forceinline__ void rank_short(const uint16_t* qu, const WindowRows& rows, int n_win,
                                           const uint16_t* ku, int len, int keep, float sm_scale,
                                           const SelectExtras& ex, float* logits, RankShortLds& lds,
                                           int32_t* idx) {
  constexpr int kWaves = THREADS / 64;
  constexpr int kPer = (kShortLen + THREADS - 1) / THREADS;  // keys per thread
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = lane & 15, g = lane >> 4;
  const int n_group = (len + 31) / 32;

  // ---- logits of every key against the window rows, and per 32 keys the maximum and sum of
  // exponentials of every window row
  {
    score_bf16x8 qf[D / 32];
    score_load_window<D>(qu, rows, n_win, qf);
    score_bf16x8 kf[2][D / 32];
    if (wave < n_group) score_load_keys<D, 2>(ku, 32 * wave, len, kf);
    for (int group = wave; group < n_group; group += kWaves) {
      score_f32x4 c[2];
      float m, e;
      score_products<D, 2>(kf, qf, c);
      if (group + kWaves < n_group) score_load_keys<D, 2>(ku, 32 * (group + kWaves), len, kf);
      score_statistics<2>(c, 32 * group, len, sm_scale, m, e);
      score_store_logits<2, true>(c, 32 * group, len, logits, kLogitStride);
      if (lane < kMaxWindow) {
        lds.group_max[group][lane] = m;
        lds.group_sum[group][lane] = e;
      }
    }
    for (int b = tid; b < 4 * 256; b += THREADS) lds.hist[b] = 0;
  }
  __syncthreads();

  // ---- row normalisers, by every wave: lane (g, i) merges virtual waves 4g .. 4g+3 of row i
  float own_shift;
  {
    float vm[4], ve[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int group = 4 * g + x;
      const float m = lds.group_max[min(group, n_group - 1)][i], e = lds.group_sum[min(group, n_group - 1)][i];
      vm[x] = group < n_group ? m : -INFINITY;
      ve[x] = group < n_group ? e : 0.f;
    }
#pragma unroll
    for (int first = kVirtualWaves; first < kShortGroups; first += kVirtualWaves)
      if (first < n_group) {  // (the same for all lanes)
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const int group = first + 4 * g + x;
          const float m = lds.group_max[min(group, n_group - 1)][i], e = lds.group_sum[min(group, n_group - 1)][i];
          if (group < n_group) join_keys(vm[x], ve[x], m, e);
        }
      }
    own_shift = row_shift<false>(vm, ve, (min(n_group, kVirtualWaves) + 3) / 4);
  }

  if constexpr (!EXTRAS) {  // few rows: several lanes to a row
    const int part4 = min(tid / 4, len - 1), part2 = min(tid / 2, len - 1);
    if (len <= THREADS / 4) {
      const float own = log_sum_parts<4>(logits + part4 * kLogitStride, n_win, own_shift);
      if (select_by_rank<THREADS, 4>(own, len, keep, lds, lds.list, idx)) return;
    } else if (len <= kCountedRows && len <= THREADS / 2) {
      const float own = log_sum_parts<2>(logits + part2 * kLogitStride, n_win, own_shift);
      if (select_by_rank<THREADS, 2>(own, len, keep, lds, lds.list, idx)) return;
    }
  }

  // ---- log-scores, as keys whose order is theirs
  float shift[kMaxWindow];
  row_shifts(own_shift, shift);
  float own[kPer];
#pragma unroll
  for (int c = 0; c < kPer; ++c) {
    const int key = tid + c * THREADS;
    if (key < len) {
      const float* lg = logits + key * kLogitStride;
      float la[kMaxWindow];
#pragma unroll
      for (int j4 = 0; j4 < kMaxWindow; j4 += 4) {
        const float4 x = *(const float4*)(lg + j4);
        la[j4] = x.x; la[j4 + 1] = x.y; la[j4 + 2] = x.z; la[j4 + 3] = x.w;
      }
      own[c] = log_sum_rows(la, n_win, shift);
    }
  }
  select_scores<THREADS, kPer, EXTRAS>(own, len, keep, ex, lds, lds.list, idx);
}

// ---- longer caches, 1024 threads, up to 1024 PER rows (PER = 4 or 12): the logits of the first rows stay
// in registers (a wave's groups of 32 keys, one per round of 512; eight rounds, or six where rows
// beyond them have to be provided for) until the row normalisers are known, and are then turned
// through a piece of LDS per wave, two groups at a time, so that a lane has the sixteen logits of one
// key.  Later rows go through the workspace.  Keeping them saves 64 bytes
// written and read per key (more than an XCD's L2 holds for 32 units of 3350 keys) and their latency.
// Bound by the HBM where there is a unit per compute unit, by the exponentials (two per key and
// window row, through one compute unit's vector pipes) where there are fewer.
constexpr int kLongInRegisters = 8 * 512;  // rows of PER = 4
constexpr int kLongTurnBytes = 16 * 64 * kLogitStride * 4;  // dynamic LDS; afterwards the index list is there
constexpr int kLongMaxPer = 12;
static_assert(kLongInRegisters == 4 * 1024 && kLongMaxPer * 1024 * 4 <= kLongTurnBytes, "the index list fits");

template <int PER>
struct RankLongLds {
  __attribute__((aligned(16))) uint32_t hist[4 * 256];
  float wave_rowmax[16][kMaxWindow], wave_rowsum[16][kMaxWindow];
  uint32_t keys[PER * 1024];
  uint32_t wave_max[16], wave_min[16];
  uint32_t count[PER * 32];  // as in RankShortLds
};

// Returns the index list (LDS, in place of `turn`).  logits_far: [len][kMaxWindow] of the unit.
template <int D, int PER, bool EXTRAS>
__device__ __forceinline__ const int32_t* rank_long(const uint16_t* qu, const WindowRows& rows, int n_win,
                                                    const uint16_t* ku, int len, int keep, float sm_scale,
                                                    const SelectExtras& ex, float* turn, float* logits_far,
                                                    RankLongLds<PER>& lds, int32_t* idx) {
  constexpr int kThreads = 1024;
  constexpr bool kFar = PER > 4;
  constexpr int kLongRounds = kFar ? 6 : 8;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = lane & 15, g = lane >> 4;
  score_f32x4 c[kLongRounds][2];
  float m_run = -INFINITY, e_run = 0.f;
  {
    score_bf16x8 qf[D / 32], kf[2][D / 32];
    score_load_window<D>(qu, rows, n_win, qf);
    if (32 * wave < len) score_load_keys<D, 2>(ku, 32 * wave, len, kf);
#pragma unroll
    for (int r = 0; r < kLongRounds; ++r) {
      const int key0 = 512 * r + 32 * wave;
      if (key0 < len) {
        score_products<D, 2>(kf, qf, c[r]);
        __builtin_amdgcn_sched_barrier(0);
        if ((kFar || r + 1 < kLongRounds) && key0 + 512 < len) score_load_keys<D, 2>(ku, key0 + 512, len, kf);
        __builtin_amdgcn_sched_barrier(0);
        float m, e;
        score_statistics<2>(c[r], key0, len, sm_scale, m, e);
        join_keys(m_run, e_run, m, e);
      }
    }
    if constexpr (kFar) {
      for (int key0 = kLongRounds * 512 + 32 * wave; key0 < len; key0 += 512) {
        score_f32x4 far[2];
        score_products<D, 2>(kf, qf, far);
        __builtin_amdgcn_sched_barrier(0);
        if (key0 + 512 < len) score_load_keys<D, 2>(ku, key0 + 512, len, kf);
        __builtin_amdgcn_sched_barrier(0);
        float m, e;
        score_statistics<2>(far, key0, len, sm_scale, m, e);
        score_store_logits<2, true>(far, key0, len, logits_far, kMaxWindow);
        join_keys(m_run, e_run, m, e);
      }
    }
  }
  if (lane < kMaxWindow) {
    lds.wave_rowmax[wave][lane] = m_run;
    lds.wave_rowsum[wave][lane] = e_run;
  }
  lds.hist[tid] = 0;
  __syncthreads();  // also makes the far logits visible to the whole workgroup
  float shift[kMaxWindow];
  {
    float vm[4], ve[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      vm[x] = lds.wave_rowmax[4 * g + x][i];
      ve[x] = lds.wave_rowsum[4 * g + x][i];
    }
    row_shifts(row_shift<true>(vm, ve, 4), shift);
  }
  auto log_score = [&](const float* lg) -> float {
    float la[kMaxWindow];
#pragma unroll
    for (int j4 = 0; j4 < kMaxWindow; j4 += 4) {
      const float4 x = *(const float4*)(lg + j4);
      la[j4] = x.x; la[j4 + 1] = x.y; la[j4 + 2] = x.z; la[j4 + 3] = x.w;
    }
    return log_sum_rows(la, n_win, shift);
  };
  float* const mine = turn + wave * (64 * kLogitStride);
  float* const raw = reinterpret_cast<float*>(lds.keys);
#pragma unroll
  for (int r = 0; r < kLongRounds; r += 2) {
    if (512 * r + 32 * wave < len) {
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int v = 0; v < 4; ++v) mine[(32 * x + 16 * t + 4 * g + v) * kLogitStride + i] = c[r + x][t][v];
      const int key = 512 * (r + (lane >> 5)) + 32 * wave + (lane & 31);
      const float ls = log_score(mine + lane * kLogitStride);
      if (key < len) raw[key] = ls;
    }
  }
  if constexpr (kFar)
    for (int key = kLongRounds * 512 + tid; key < len; key += kThreads)
      raw[key] = log_score(logits_far + (long long)key * kMaxWindow);
  __syncthreads();
  float own[PER];
#pragma unroll
  for (int x = 0; x < PER; ++x)
    if (tid + x * kThreads < len) own[x] = raw[tid + x * kThreads];
  __syncthreads();
  int32_t* const list = reinterpret_cast<int32_t*>(turn);
  select_scores<kThreads, PER, EXTRAS>(own, len, keep, ex, lds, list, idx);
  return list;
}

}  // namespace scalekv
