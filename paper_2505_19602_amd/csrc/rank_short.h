// Ranking of one unit's short cache by one workgroup (Eq. 5 and the top-k of Sec. 3.3, bf16), all
// of it in registers and LDS: logits, row normalisers, log-scores, selection, index list.
//
// At these lengths nothing is bound by bandwidth; the time is a chain of memory latencies and
// barriers.  Against the general ranking kernel (select.hip) the chain is shorter by the round
// trip of the logits through global memory (they stay in LDS, 80 bytes a key: 16 window rows and a
// pad against bank conflicts), by the hand-over of the row normalisers (every wave forms them
// itself) and by the radix passes over bits that all keys share or that no longer matter: the
// first digit starts at the highest bit in which the largest and the smallest key differ, and the
// search ends as soon as the digit's bin is wanted whole.
//
// The arithmetic is that of select.hip, operation by operation (groups of 32 keys belong to
// virtual waves group % 16, whose running maximum and sum are merged in group order, then in wave
// order), so the two kernels select the same rows bit for bit.
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
  uint32_t count[2 * kShortLen / 64];       // per 64 keys: above the threshold, equal to it
};
// dynamic LDS for the logits
inline int rank_short_logit_bytes(int len) { return round_up(len, 32) * kLogitStride * 4; }

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
    for (int group = wave; group < n_group; group += kWaves) {
      float m, e;
      score_wave_logits<D, 2>(ku, qf, 32 * group, len, sm_scale, logits, kLogitStride, m, e);
      if (lane < kMaxWindow) {
        lds.group_max[group][lane] = m;
        lds.group_sum[group][lane] = e;
      }
    }
    for (int b = tid; b < 4 * 256; b += THREADS) lds.hist[b] = 0;
  }
  __syncthreads();

  // ---- row normalisers, by every wave: lane (g, i) merges virtual waves 4g .. 4g+3 of row i
  float shift[kMaxWindow];
  {
    float vm[4], ve[4];
    float mm = -INFINITY;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      float m_run = -INFINITY, e_run = 0.f;
      for (int group = 4 * g + x; group < n_group; group += kVirtualWaves) {
        const float m = lds.group_max[group][i], e = lds.group_sum[group][i];
        const float m_new = fmaxf(m_run, m);
        e_run = e_run * expf(m_run - m_new) + e * expf(m - m_new);
        m_run = m_new;
      }
      vm[x] = m_run;
      ve[x] = e_run;
      mm = fmaxf(mm, m_run);
    }
    mm = xor32_max(xor16_max(mm));
    // the sum runs over the virtual waves in order: g = 0 hands its part to g = 1 and so on
    float z = 0.f;
#pragma unroll
    for (int turn = 0; turn < 4; ++turn) {
      float part = z;
#pragma unroll
      for (int x = 0; x < 4; ++x)
        if (vm[x] > -INFINITY) part += ve[x] * expf(vm[x] - mm);
      // after turn t the lanes of g = t hold the sum so far; everybody takes it from there
      z = __shfl(part, 16 * turn + i);
    }
    const float s = mm + logf(z);
#pragma unroll
    for (int j = 0; j < kMaxWindow; ++j)
      shift[j] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(s), j));
  }

  // ---- log-scores, as keys whose order is theirs
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
  if constexpr (EXTRAS) {
    if (ex.pool_w > 1) {
      float* raw = reinterpret_cast<float*>(lds.keys);
#pragma unroll
      for (int c = 0; c < kPer; ++c)
        if (tid + c * THREADS < len) raw[tid + c * THREADS] = own[c];
      __syncthreads();
#pragma unroll
      for (int c = 0; c < kPer; ++c)
        if (tid + c * THREADS < len)
          own[c] = pooled_log([&](int t) { return raw[t]; }, tid + c * THREADS, len, (ex.pool_w - 1) / 2);
      __syncthreads();
    }
  }
  uint32_t kk[kPer];
  uint32_t hi = 0, lo = 0xffffffffu;
#pragma unroll
  for (int c = 0; c < kPer; ++c) {
    const int key = tid + c * THREADS;
    kk[c] = 0;
    if (key < len) {
      kk[c] = order_key(own[c]);
      if constexpr (EXTRAS) {
        for (int j = 0; j < ex.n_forced; ++j)
          if (ex.forced[j] == key) kk[c] = 0xffffffffu;
      }
      lds.keys[key] = kk[c];
      hi = max(hi, kk[c]);
      lo = min(lo, kk[c]);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, off));
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, off));
  }
  if (lane == 0) { lds.wave_max[wave] = hi; lds.wave_min[wave] = lo; }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    hi = max(hi, lds.wave_max[w]);
    lo = min(lo, lds.wave_min[w]);
  }

  // ---- threshold: keys above T are selected, and the first need_eq of those equal to it
  uint32_t T, need_eq;
  radix_kth_largest_from<THREADS>([&](int t) { return lds.keys[t]; }, len, (uint32_t)keep,
                                  32 - __builtin_clz((hi ^ lo) | 1u), hi, lds.hist, T, need_eq);

  // ---- positions in ascending order of the rows: 64 rows per entry of lds.count
  const int n_slot = (len + 63) / 64;
#pragma unroll
  for (int c = 0; c < kPer; ++c) {
    const int slot = c * kWaves + wave;
    if (slot < n_slot) {
      const bool valid = tid + c * THREADS < len;
      const uint32_t gt = __builtin_popcountll(__builtin_amdgcn_ballot_w64(valid && kk[c] > T));
      const uint32_t eq = __builtin_popcountll(__builtin_amdgcn_ballot_w64(valid && kk[c] == T));
      if (lane == 0) lds.count[slot] = gt | eq << 16;
    }
  }
  __syncthreads();
  const uint32_t mine = lane < n_slot ? lds.count[lane] : 0u;  // (n_slot <= 24; both halves stay below 2^16)
  const uint32_t before = wave_prefix_sum(mine, lane) - mine;
#pragma unroll
  for (int c = 0; c < kPer; ++c) {
    const int slot = c * kWaves + wave;
    if (slot < n_slot) {
      const uint32_t base = __builtin_amdgcn_readlane(before, slot);
      const int key = tid + c * THREADS;
      const bool valid = key < len;
      const unsigned long long gt = __builtin_amdgcn_ballot_w64(valid && kk[c] > T);
      const unsigned long long eq = __builtin_amdgcn_ballot_w64(valid && kk[c] == T);
      const unsigned long long below = ((unsigned long long)1 << lane) - 1;
      const uint32_t g_before = (base & 0xffffu) + __builtin_popcountll(gt & below);
      const uint32_t e_before = (base >> 16) + __builtin_popcountll(eq & below);
      const bool take = (gt >> lane & 1) || ((eq >> lane & 1) && e_before < need_eq);
      if (take) {
        const uint32_t pos = g_before + min(e_before, need_eq);
        lds.list[pos] = key;
        if (idx) idx[pos] = key;
      }
    }
  }
  __syncthreads();
}

}  // namespace scalekv
