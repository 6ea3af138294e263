// Attention Selectivity Index, Eq. 2: for sampled queries of the current map, the
// attention mass that falls on the map's own keys and the sum of the K' largest
// weights on the history keys.  Calibration-time work (the paper runs it once, on
// a handful of prompts), built on the score kernels: the logits of up to 16 query
// rows against every key are already in the workspace, key-major, with the
// per-chunk softmax statistics beside them.
//
// One workgroup per (unit, query row).  The row's normaliser comes from the chunk
// statistics; the current-map mass is a plain sum; the top-K' sum needs no sort:
// a radix select over the order-preserving images of the history logits gives the
// K'-th largest value T, and the sum is (weights above T) + (copies of T that belong
// to the top K') * weight(T) -- equal logits have equal weights, so which of them are
// taken does not matter.  All float sums run in a fixed order (strided per thread,
// butterfly per wave, waves in sequence): results do not depend on scheduling.
//
// bf16 with K' up to 256, the use the paper describes, takes a route of its own without that
// workspace of logits (asi_stream_kernel below) where there is enough of it (asi_stream_pays() in common.h).
#include "common.h"
#include "radix_select.h"
#include "score_mfma.h"

namespace scalekv {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kLdsKeys = 12288;  // history rows up to this many keep their keys in LDS

// Sum of x over the workgroup, same value in every thread.  red: kWaves floats of LDS.
__device__ __forceinline__ float block_sum(float x, float* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  __syncthreads();  // red may still be read from a previous call
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  float total = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) total += red[w];
  return total;
}

template <bool IN_LDS>
__global__ __launch_bounds__(kThreads) void asi_terms_kernel(ScoreWorkspace ws, int hist_len,
                                                             int len, int top_k,
                                                             float* __restrict__ terms, int n_samp,
                                                             int row0) {
  __shared__ uint32_t keys[IN_LDS ? kLdsKeys : 1];
  __shared__ __attribute__((aligned(16))) uint32_t hist[kRadixHistWords];
  __shared__ float red[kWaves];
  __shared__ float row_shift[kMaxWindow], stage[kStatChunks * 2 * kMaxWindow];

  const int row = SCALEKV_WG_X, unit = SCALEKV_WG_Y;
  const int tid = threadIdx.x;
  const float* lg = ws.logits + (long long)unit * ws.len_pad * kMaxWindow + row;
  auto logit = [&](int i) -> float { return lg[(long long)i * kMaxWindow]; };
  score_row_shifts(ws, unit, kMaxWindow, stage, row_shift);  // max + log Z over all `len` keys
  const float shift = row_shift[row];

  // attention mass on the current map: keys [hist_len, len)
  float part = 0.f;
  for (int i = hist_len + tid; i < len; i += kThreads) part += expf(logit(i) - shift);
  float cur = block_sum(part, red);

  // sum of the K' largest history weights
  const int kk = min(top_k, hist_len);
  float top = 0.f;
  if (kk > 0) {
    if constexpr (IN_LDS) {
      for (int i = tid; i < hist_len; i += kThreads) keys[i] = order_key(logit(i));
      __syncthreads();
    }
    auto key_at = [&](int i) -> uint32_t {
      if constexpr (IN_LDS) return keys[i];
      else return order_key(logit(i));
    };
    uint32_t T = 0, need_eq = 0;
    if (kk < hist_len) radix_kth_largest<kThreads>(key_at, hist_len, (uint32_t)kk, hist, T, need_eq);
    part = 0.f;
    for (int i = tid; i < hist_len; i += kThreads) {
      const uint32_t key = key_at(i);
      if (kk == hist_len || key > T || order_key_is_nan(key)) part += expf(order_key_value(key) - shift);
    }
    top = block_sum(part, red);
    if (kk < hist_len) top += (float)need_eq * expf(order_key_value(T) - shift);
    // a key of NaN makes the row NaN (the normaliser passes over one that is alone among its 64 keys)
    if (cur != cur || top != top) cur = top = cur + top;
  }
  if (tid == 0) {
    float* out = terms + ((long long)unit * n_samp + row0 + row) * 2;
    out[0] = cur;
    out[1] = top;
  }
}

// ---- bf16, top_k <= kStreamTopK: the keys are read once and their logits never leave the chip.
//
// One workgroup per unit and part of its keys, 16 waves x 32 keys per round, 16 NB query rows.  A
// lane keeps running softmax sums of its own (history and current map apart) and compares its
// history logits with the row's threshold, a lower bound of the K'-th largest so far; what is above
// is appended to the row's candidates in LDS.  When a row's list could overflow in the next round
// (in the first two or three rounds; then the threshold admits K' / n of the keys), every wave cuts
// the lists of its rows down to their K' largest and raises the threshold.  What is left at the end,
// K' values a row, goes to the workspace with the sums; asi_merge_kernel joins the parts.
// The order in which candidates arrive is not fixed, the multiset of the K' largest is, and its
// weights are added as integers (2^-40 of the largest): results are reproducible bit for bit.
// Bound by HBM: the keys once.  256 units x 10585 keys, 16 rows, K' = 64: 139 us, 5.0 TB/s
// (logits through the workspace and one radix select per row: 159 + 416 us).
constexpr int kStreamTopK = 256;
constexpr int kListCap = 1024;                     // candidates per row; a round adds at most kRoundKeys
constexpr int kRoundKeys = kWaves * 32;
constexpr int kListLimit = kListCap - kRoundKeys;  // cut down above this
static_assert(kListLimit >= kStreamTopK, "a list that has been cut down has room for a round");

// Cuts the n values of one row's list down to their k largest (any order), by one wave.  Returns a
// lower bound below which no further value can be among the k largest.
__device__ __forceinline__ float cut_list(float* list, int n, int k) {
  constexpr int kPer = kListCap / 64;
  const int lane = threadIdx.x & 63;
  uint32_t key[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) key[j] = 64 * j + lane < n ? order_key(list[64 * j + lane]) : 0u;
  // the largest T with at least k keys >= T, bit by bit; done early if exactly k remain
  uint32_t T = 0;
  int count = n;
  for (int bit = 31; bit >= 0 && count != k; --bit) {
    const uint32_t cand = T | 1u << bit;
    int c = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) c += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key[j] >= cand));
    if (c >= k) { T = cand; count = c; }
  }
  int extra = count - k;  // copies of T beyond the k largest
  int base = 0;
  const unsigned long long below = ((unsigned long long)1 << lane) - 1;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const unsigned long long eq = __builtin_amdgcn_ballot_w64(key[j] == T);
    const bool drop = key[j] == T && __builtin_popcountll(eq & below) < extra;
    const bool take = key[j] >= T && !drop && 64 * j + lane < n;
    const unsigned long long m = __builtin_amdgcn_ballot_w64(take);
    if (take) list[base + __builtin_popcountll(m & below)] = order_key_value(key[j]);
    base += __builtin_popcountll(m);
    extra = max(0, extra - (int)__builtin_popcountll(eq));
  }
  return T ? order_key_value(T - 1) : -INFINITY;
}

struct AsiStream {
  const uint16_t* q;
  long long q_unit_stride;
  int row0, n_rows;
  const uint16_t* k;
  long long k_seq_stride, k_head_stride;
  int n_head, hist_len, len, part_len, n_part, top_k;
  float scale_log2e;
  float* stats;  // [U][n_part][3][16 NB]: maximum (scaled, log2 units), sum over history, sum over the map
  float* cand;   // [U][n_part][16 NB][top_k] raw logits, padded with -inf
};

template <int D, int NB>
__global__ __launch_bounds__(kThreads) void asi_stream_kernel(AsiStream a) {
  constexpr int NSL = D / 32, kRows = 16 * NB;
  extern __shared__ float lists[];  // [kRows][kListCap]
  __shared__ int count[kRows];
  __shared__ float threshold[kRows];
  __shared__ int full[4];           // by round % 4: some list is above kListLimit
  __shared__ float red[3][kWaves][kRows];
  const int unit = SCALEKV_WG_Y, part = SCALEKV_WG_X;
  const int seq = unit / a.n_head, head = unit - seq * a.n_head;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = lane & 15, g = lane >> 4;
  const uint16_t* ku = a.k + seq * a.k_seq_stride + head * a.k_head_stride;
  const int begin = part * a.part_len, end = min(begin + a.part_len, a.len);
  const bool lists_on = a.top_k > 0 && a.top_k < a.hist_len;  // otherwise nothing to choose

  if (tid < kRows) { count[tid] = 0; threshold[tid] = -INFINITY; }
  if (tid < 4) full[tid] = 0;
  score_bf16x8 qf[NB][NSL];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int row = a.row0 + min(16 * b + i, a.n_rows - 1);  // rows past the end repeat the last and are not used
#pragma unroll
    for (int sl = 0; sl < NSL; ++sl)
      qf[b][sl] = *(const score_bf16x8*)(a.q + unit * a.q_unit_stride + (long long)row * D + 32 * sl + 8 * g);
  }
  score_bf16x8 kf[2][NSL];
  auto load = [&](int key0) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const uint16_t* row = ku + (long long)min(key0 + 16 * t + i, a.len - 1) * D + 8 * g;
#pragma unroll
      for (int sl = 0; sl < NSL; ++sl) kf[t][sl] = *(const score_bf16x8*)(row + 32 * sl);
    }
  };
  float m[NB], eh[NB], ec[NB], thr[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) { m[b] = -INFINITY; eh[b] = 0.f; ec[b] = 0.f; thr[b] = -INFINITY; }
  load(begin + 32 * wave);
  __syncthreads();

  int round = 0;
  for (int base = begin; base < end; base += kRoundKeys, ++round) {
    const int key0 = base + 32 * wave;
    score_f32x4 c[NB][2];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        c[b][t] = score_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl)
          c[b][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[t][sl], qf[b][sl], c[b][t], 0, 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
    if (base + kRoundKeys < end) load(key0 + kRoundKeys);
    __builtin_amdgcn_sched_barrier(0);
    if (key0 < end) {
      // register v of tile t is key key0 + 16t + 4g + v
      const int own = key0 + 4 * g;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        float top = m[b];
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const bool in = own + 16 * (x / 4) + x % 4 < end;
          c[b][x / 4][x % 4] = in ? c[b][x / 4][x % 4] : -INFINITY;
          top = fmaxf(top, c[b][x / 4][x % 4] * a.scale_log2e);
        }
        if (top > -INFINITY) {
          const float alpha = __builtin_amdgcn_exp2f(m[b] - top);
          float h = 0.f, u = 0.f;
#pragma unroll
          for (int x = 0; x < 8; ++x) {
            const float w = __builtin_amdgcn_exp2f(fmaf(c[b][x / 4][x % 4], a.scale_log2e, -top));
            const bool hist = own + 16 * (x / 4) + x % 4 < a.hist_len;
            h += hist ? w : 0.f;
            u += hist ? 0.f : w;
          }
          eh[b] = fmaf(eh[b], alpha, h);
          ec[b] = fmaf(ec[b], alpha, u);
          m[b] = top;
        } else {  // nothing but -inf and NaN (the maximum passes over NaN; the sums do not)
#pragma unroll
          for (int x = 0; x < 8; ++x)
            if (c[b][x / 4][x % 4] != c[b][x / 4][x % 4]) eh[b] = c[b][x / 4][x % 4];
        }
      }
      if (lists_on && key0 < a.hist_len) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          bool take[8];
          int n = 0;
#pragma unroll
          for (int x = 0; x < 8; ++x) {
            take[x] = own + 16 * (x / 4) + x % 4 < min(end, a.hist_len) && !(c[b][x / 4][x % 4] <= thr[b]);
            n += take[x];
          }
          if (n > 0) {
            int pos = atomicAdd(&count[16 * b + i], n);
            if (pos + n > kListLimit) full[round & 3] = 1;
            float* list = lists + (16 * b + i) * kListCap;
#pragma unroll
            for (int x = 0; x < 8; ++x)
              if (take[x]) list[pos++] = c[b][x / 4][x % 4];
          }
        }
      }
    }
    __syncthreads();
    // (the flag of round + 2 is cleared here: nobody sets it before passing the next barrier)
    if (tid == 0) full[(round + 2) & 3] = 0;
    if (full[round & 3]) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int row = 16 * b + wave, n = count[row];
        if (n > a.top_k) {
          const float t = cut_list(lists + row * kListCap, n, a.top_k);
          if (lane == 0) { count[row] = a.top_k; threshold[row] = t; }
        }
      }
      __syncthreads();
#pragma unroll
      for (int b = 0; b < NB; ++b) thr[b] = threshold[16 * b + i];
    }
  }

  // ---- sums: lanes of a row, then the waves in order
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const float top = xor32_max(xor16_max(m[b]));
    const float f = m[b] > -INFINITY ? __builtin_amdgcn_exp2f(m[b] - top) : 0.f;
    const float h = xor32_sum(xor16_sum(eh[b] * f)), u = xor32_sum(xor16_sum(ec[b] * f));
    if (g == 0) { red[0][wave][16 * b + i] = top; red[1][wave][16 * b + i] = h; red[2][wave][16 * b + i] = u; }
  }
  __syncthreads();
  float* stats = a.stats + ((long long)unit * a.n_part + part) * 3 * kRows;
  if (tid < kRows) {
    float top = -INFINITY;
    for (int w = 0; w < kWaves; ++w) top = fmaxf(top, red[0][w][tid]);
    float h = 0.f, u = 0.f;
    for (int w = 0; w < kWaves; ++w) {
      const float f = red[0][w][tid] > -INFINITY ? __builtin_amdgcn_exp2f(red[0][w][tid] - top) : 0.f;
      h = fmaf(red[1][w][tid], f, h);
      u = fmaf(red[2][w][tid], f, u);
    }
    stats[tid] = top;
    stats[kRows + tid] = h;
    stats[2 * kRows + tid] = u;
  }
  if (!lists_on) return;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int row = 16 * b + wave;
    float* list = lists + row * kListCap;
    const int n = count[row];
    if (n > a.top_k) cut_list(list, n, a.top_k);
    float* out = a.cand + (((long long)unit * a.n_part + part) * kRows + row) * a.top_k;
    for (int x = lane; x < a.top_k; x += 64) out[x] = x < n ? list[x] : -INFINITY;
  }
}

// Joins the parts of one (unit, query row): sums in order, the K' largest of all candidates.
constexpr int kMergeThreads = 256;
constexpr int kMaxParts = 16;
__global__ __launch_bounds__(kMergeThreads) void asi_merge_kernel(AsiStream a, int rows_per_pass, float* __restrict__ terms,
                                                                  int n_samp) {
  __shared__ uint32_t keys[kMaxParts * kStreamTopK];
  __shared__ __attribute__((aligned(16))) uint32_t hist[kRadixHistWords];
  __shared__ uint32_t wave_top[kMergeThreads / 64];
  __shared__ unsigned long long wave_sum[kMergeThreads / 64];
  const int row = SCALEKV_WG_X, unit = SCALEKV_WG_Y, tid = threadIdx.x;
  const float* stats = a.stats + (long long)unit * a.n_part * 3 * rows_per_pass + row;
  float top = -INFINITY;
  for (int p = 0; p < a.n_part; ++p) top = fmaxf(top, stats[p * 3 * rows_per_pass]);
  float h = 0.f, u = 0.f;
  for (int p = 0; p < a.n_part; ++p) {
    const float mp = stats[p * 3 * rows_per_pass];
    const float f = mp > -INFINITY ? __builtin_amdgcn_exp2f(mp - top) : 0.f;
    h = fmaf(stats[(p * 3 + 1) * rows_per_pass], f, h);
    u = fmaf(stats[(p * 3 + 2) * rows_per_pass], f, u);
  }
  const float z = h + u;
  float best = 0.f;
  if (a.top_k >= a.hist_len) {
    best = h / z;  // every history row (none: 0)
  } else if (a.top_k > 0) {
    const int n = a.n_part * a.top_k;
    uint32_t largest = 0;
    for (int x = tid; x < n; x += kMergeThreads) {
      const int p = x / a.top_k, j = x - p * a.top_k;
      keys[x] = order_key(a.cand[(((long long)unit * a.n_part + p) * rows_per_pass + row) * a.top_k + j]);
      largest = max(largest, keys[x]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) largest = max(largest, (uint32_t)__shfl_xor((int)largest, off));
    if ((tid & 63) == 0) wave_top[tid >> 6] = largest;
    __syncthreads();
    for (int w = 0; w < kMergeThreads / 64; ++w) largest = max(largest, wave_top[w]);
    uint32_t T = 0, need_eq = 0;  // everything counts
    if (a.n_part > 1)
      radix_kth_largest<kMergeThreads>([&](int x) { return keys[x]; }, n, (uint32_t)a.top_k, hist, T, need_eq);
    const float lead = order_key_value(largest);
    auto weight = [&](uint32_t key) -> unsigned long long {  // of the largest, in 2^-40
      return (unsigned long long)(__builtin_amdgcn_exp2f((order_key_value(key) - lead) * a.scale_log2e) * 0x1p40f);
    };
    unsigned long long sum = 0;
    for (int x = tid; x < n; x += kMergeThreads)
      if (keys[x] > T) sum += weight(keys[x]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if ((tid & 63) == 0) wave_sum[tid >> 6] = sum;
    __syncthreads();
    sum = need_eq ? need_eq * weight(T) : 0;
    for (int w = 0; w < kMergeThreads / 64; ++w) sum += wave_sum[w];
    best = (float)sum * 0x1p-40f * __builtin_amdgcn_exp2f(fmaf(lead, a.scale_log2e, -top)) / z;
  }
  if (tid == 0) {
    float* out = terms + ((long long)unit * n_samp + a.row0 + row) * 2;
    out[0] = u / z;
    out[1] = best;
  }
}

template <int D, int NB>
hipError_t launch_stream(const AsiStream& a, int n_unit, float* terms, int n_samp, hipStream_t stream) {
  static std::atomic<uint64_t> configured{0};
  constexpr int kLds = 16 * NB * kListCap * 4;
  const hipError_t e = allow_dynamic_lds((const void*)asi_stream_kernel<D, NB>, kLds, configured);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((asi_stream_kernel<D, NB>), dim3(a.n_part, n_unit), dim3(kThreads), kLds, stream, a);
  hipLaunchKernelGGL(asi_merge_kernel, dim3(a.n_rows, n_unit), dim3(kMergeThreads), 0, stream, a, 16 * NB, terms,
                     n_samp);
  return hipGetLastError();
}

__global__ __launch_bounds__(kThreads) void asi_mean_kernel(const float* __restrict__ terms,
                                                            long long n, float* __restrict__ out) {
  __shared__ float red[kWaves];
  float a = 0.f, b = 0.f;
  for (long long i = threadIdx.x; i < n; i += kThreads) {
    a += terms[2 * i];
    b += terms[2 * i + 1];
  }
  const float sa = block_sum(a, red), sb = block_sum(b, red);
  if (threadIdx.x == 0) {
    const float ma = sa / (float)n, mb = sb / (float)n;
    out[0] = ma;
    out[1] = mb;
    out[2] = ma * mb;
  }
}

}  // namespace

hipError_t launch_asi_terms(int n_unit, ScoreWorkspace ws, int n_rows, int hist_len, int len,
                            int top_k, float* terms, int n_samp, int row0, hipStream_t stream) {
  if (n_unit <= 0 || n_rows <= 0 || len <= 0) return hipSuccess;
  dim3 grid(n_rows, n_unit);
  if (hist_len <= kLdsKeys)
    hipLaunchKernelGGL((asi_terms_kernel<true>), grid, dim3(kThreads), 0, stream, ws, hist_len, len,
                       top_k, terms, n_samp, row0);
  else
    hipLaunchKernelGGL((asi_terms_kernel<false>), grid, dim3(kThreads), 0, stream, ws, hist_len, len,
                       top_k, terms, n_samp, row0);
  return hipGetLastError();
}

hipError_t launch_asi_stream(int dtype, int n_seq, int n_head, int d, const void* q, int n_samp, KvView k,
                             int hist_len, int len, int top_k, float sm_scale, void* ws, size_t ws_bytes,
                             float* terms, hipStream_t stream) {
  const int n_unit = n_seq * n_head;
  if (dtype != 1 || top_k > kStreamTopK || !asi_stream_pays(n_unit, len, n_samp)) return hipErrorNotSupported;
  // parts of at least two rounds, as many as give every compute unit a workgroup
  int n_part = 1;
  while (n_part < kMaxParts && n_unit * n_part * 2 <= 256 && len >= n_part * 2 * 2 * kRoundKeys) n_part *= 2;
  AsiStream a{};
  a.q = (const uint16_t*)q;
  a.q_unit_stride = (long long)n_samp * d;
  a.k = (const uint16_t*)k.ptr; a.k_seq_stride = k.seq_stride; a.k_head_stride = k.head_stride;
  a.n_head = n_head; a.hist_len = hist_len; a.len = len; a.top_k = top_k;
  a.scale_log2e = sm_scale * 1.4426950408889634f;
  a.n_part = n_part;
  a.part_len = round_up((len + n_part - 1) / n_part, kRoundKeys);
  // 32 rows per pass over the keys, if there are that many and the workspace (sized for the logits of
  // 16 rows) holds their candidates
  const size_t per_row = (size_t)n_unit * n_part * (3 + (top_k < hist_len ? top_k : 0)) * sizeof(float);
  const int rows = n_samp > 16 && 32 * per_row <= ws_bytes ? 32 : 16;
  if (rows * per_row > ws_bytes) return hipErrorNotSupported;
  a.stats = (float*)ws;
  a.cand = a.stats + (size_t)n_unit * n_part * 3 * rows;
  for (int row0 = 0; row0 < n_samp; row0 += rows) {
    a.row0 = row0;
    a.n_rows = n_samp - row0 < rows ? n_samp - row0 : rows;
    hipError_t e;
    if (d == 128) e = rows == 32 ? launch_stream<128, 2>(a, n_unit, terms, n_samp, stream)
                                 : launch_stream<128, 1>(a, n_unit, terms, n_samp, stream);
    else e = rows == 32 ? launch_stream<64, 2>(a, n_unit, terms, n_samp, stream)
                        : launch_stream<64, 1>(a, n_unit, terms, n_samp, stream);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_asi_mean(const float* terms, long long n, float* out, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(asi_mean_kernel, dim3(1), dim3(kThreads), 0, stream, terms, n, out);
  return hipGetLastError();
}

}  // namespace scalekv
