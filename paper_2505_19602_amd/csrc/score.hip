// Importance score of Eq. 5: for every cached key i of a unit,
//   s_i = sum over window rows j of softmax_i(q_j . k_i * sm_scale),
// reported as log s_i.
//
// Two kernels.  `logits` streams the cached keys once (the HBM-bound part),
// writes the fp32 logits of the <=16 window rows (key-major, 64 B per key) and, per
// 256-key chunk, each
// row's running max and sum of exp.  `finalize` merges the chunk statistics
// into the row normalisers and folds the rows with a log-sum-exp, so no
// probability is ever rounded below fp32 and nothing underflows.
#include "common.h"
#include "score_mfma.h"

namespace scalekv {
namespace {

constexpr int kThreads = kScoreChunk;  // 64 keys per wave

typedef score_f32x4 f32x4;

// Row maxima and sums of exponentials of a chunk from those of its waves.
__device__ __forceinline__ void store_chunk_statistics(const float (&red_max)[kThreads / 64][kMaxWindow],
                                                       const float (&red_sum)[kThreads / 64][kMaxWindow],
                                                       const ScoreWorkspace& ws, int unit) {
  const int tid = threadIdx.x;
  if (tid >= kMaxWindow) return;
  float m = -INFINITY;
  for (int w = 0; w < kThreads / 64; ++w) m = fmaxf(m, red_max[w][tid]);
  float sum = 0.f;
  for (int w = 0; w < kThreads / 64; ++w)
    if (red_max[w][tid] > -INFINITY) sum += red_sum[w][tid] * expf(red_max[w][tid] - m);
  float* part = ws.partial + ((long long)unit * ws.n_chunk + SCALEKV_WG_X) * 2 * kMaxWindow;
  part[tid] = m;
  part[kMaxWindow + tid] = sum;
}

// fp32 logits kernel, on MFMA 16x16x4, whose four products are added one after the other, each sum rounded: the logits
// have the bits of a chain of fma in channel order (468 shapes and value ranges, with denormals and infinities, compared
// with such a kernel).  A wave takes 64 keys, as four tiles, and all its key vectors are requested at once: a launch of a
// few rows is bound by the latencies one after the other.  Both operands arrive as 16 bytes per lane, channels 16t + 4g .. +3 of a row in lane (g, i): a 4 x 4 transposition
// over the lane groups, four swaps, makes of them the operands of four steps, channels 16t + 4s + g of step s.
// Before, a thread per key and four rows, keys through LDS 32 channels at a time, queries as scalars, a wait for every
// few of them; whole steps, us, so / now (d 128): 80 units x 30 keys 21.5 / 18.1, 32 x 585, 400 queries 81.0 / 78.3, 64 x 1200
// 52 / 44.5, 256 x 800 92 / 75.2.
template <int D>
__device__ __forceinline__ void load_steps_f32(const float* row, f32x4 (&x)[D / 16]) {
  const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int t = 0; t < D / 16; ++t) x[t] = *(const f32x4*)(row + 16 * t + 4 * g);
}
// [element of lane group g] -> [step], element e of group g becoming step g of group e
__device__ __forceinline__ void transpose_groups(f32x4& x) {
  auto swap32 = [](float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  };
  auto swap16 = [](float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  };
  float x0 = x[0], x1 = x[1], x2 = x[2], x3 = x[3];
  swap32(x0, x2);
  swap32(x1, x3);
  swap16(x0, x1);
  swap16(x2, x3);
  x = f32x4{x0, x1, x2, x3};
}
template <int D>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 2))) void score_logits_f32_kernel(
    const float* __restrict__ q, long long q_unit_stride, WindowRows rows, int n_win,
    const float* __restrict__ k, long long k_seq_stride, long long k_head_stride, int n_head,
    int cache_len, float sm_scale, ScoreWorkspace ws) {
  constexpr int NT = 4, NV = D / 16;
  __shared__ float red_max[kThreads / 64][kMaxWindow], red_sum[kThreads / 64][kMaxWindow];
  const int unit = SCALEKV_WG_Y;
  const int seq = unit / n_head, head = unit - seq * n_head;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = lane & 15, g = lane >> 4;
  const int key0 = SCALEKV_WG_X * kScoreChunk + wave * (16 * NT);
  const float* ku = k + seq * k_seq_stride + head * k_head_stride;
  if (key0 < cache_len) {
    f32x4 kf[NT][NV], qf[NV], c[NT];
    int row = 0;  // (as in score_load_window; rows from n_win on are never used)
#pragma unroll
    for (int j = 0; j < kMaxWindow; ++j) row = i == j ? rows.row[j] : row;
    load_steps_f32<D>(q + unit * q_unit_stride + (long long)row * D, qf);
#pragma unroll
    for (int t = 0; t < NT; ++t)  // clamp: legal address, value unused
      load_steps_f32<D>(ku + (long long)min(key0 + 16 * t + i, cache_len - 1) * D, kf[t]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int x = 0; x < NV; ++x) transpose_groups(qf[x]);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      c[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int x = 0; x < NV; ++x) transpose_groups(kf[t][x]);
    }
#pragma unroll
    for (int x = 0; x < NV; ++x)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t) c[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][x][s], qf[x][s], c[t], 0, 0, 0);
    // register v of tile t: key key0 + 16t + 4g + v against window row i
    float m = -INFINITY;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const bool valid = key0 + 16 * t + 4 * g + v < cache_len;
        c[t][v] = valid ? c[t][v] * sm_scale : -INFINITY;
        m = fmaxf(m, c[t][v]);
      }
    m = xor32_max(xor16_max(m));
    score_store_logits<NT, true>(c, key0, cache_len, ws.logits + (long long)unit * ws.len_pad * kMaxWindow, kMaxWindow);
    // the exponentials are added key k to k + 32, then + 16, + 8, + 4, + 2, + 1
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) c[t][v] = key0 + 16 * t + 4 * g + v < cache_len ? expf(c[t][v] - m) : 0.f;
    f32x4 e = (c[0] + c[2]) + (c[1] + c[3]);
#pragma unroll
    for (int v = 0; v < 4; ++v) e[v] = xor16_sum(xor32_sum(e[v]));
    const float sum = (e[0] + e[2]) + (e[1] + e[3]);
    if (lane < kMaxWindow) { red_max[wave][lane] = m; red_sum[wave][lane] = sum; }
  } else if (lane < kMaxWindow) {
    red_max[wave][lane] = -INFINITY;
    red_sum[wave][lane] = 0.f;
  }
  __syncthreads();
  store_chunk_statistics(red_max, red_sum, ws, unit);
}

// bf16 logits kernel: the HBM-bound part of the score.  Each wave handles 64 keys of the
// workgroup's 256-key chunk (see score_mfma.h) and the workgroup leaves the chunk's row maximum
// and sum of exponentials for the finalisation.
template <int D>
__global__ __launch_bounds__(kThreads) void score_logits_mfma_kernel(
    const uint16_t* __restrict__ q, long long q_unit_stride, WindowRows rows, int n_win,
    const uint16_t* __restrict__ k, long long k_seq_stride, long long k_head_stride, int n_head,
    int cache_len, float sm_scale, ScoreWorkspace ws) {
  constexpr int NT = 4;  // 16-key tiles per wave
  __shared__ float red_max[kThreads / 64][kMaxWindow];
  __shared__ float red_sum[kThreads / 64][kMaxWindow];
  const int unit = SCALEKV_WG_Y;
  const int seq = unit / n_head, head = unit - seq * n_head;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint16_t* ku = k + seq * k_seq_stride + head * k_head_stride;
  score_bf16x8 qf[D / 32];
  score_load_window<D>(q + unit * q_unit_stride, rows, n_win, qf);
  float m, e;
  score_wave_logits<D, NT>(ku, qf, SCALEKV_WG_X * kScoreChunk + wave * (16 * NT), cache_len, sm_scale,
                           ws.logits + (long long)unit * ws.len_pad * kMaxWindow, kMaxWindow, m, e);
  if (lane < kMaxWindow) { red_max[wave][lane] = m; red_sum[wave][lane] = e; }
  __syncthreads();
  store_chunk_statistics(red_max, red_sum, ws, unit);
}

// log s_i = logsumexp_j( logit[j][i] - max_j - log Z_j ).
__global__ __launch_bounds__(256) void score_finalize_kernel(int n_win, int cache_len,
                                                             ScoreWorkspace ws,
                                                             float* __restrict__ log_scores,
                                                             long long score_unit_stride) {
  __shared__ float row_shift[kMaxWindow], stage[kStatChunks * 2 * kMaxWindow];
  const int unit = SCALEKV_WG_Y;
  const int tid = threadIdx.x;
  score_row_shifts(ws, unit, n_win, stage, row_shift);
  const int key = SCALEKV_WG_X * 256 + tid;
  if (key >= cache_len) return;
  log_scores[unit * score_unit_stride + key] = score_log_sum(ws, unit, key, n_win, row_shift);
}

}  // namespace

hipError_t launch_score_logits(int dtype, int n_seq, int n_head, int d, const void* q,
                               long long q_unit_stride, WindowRows rows, int n_win, KvView k,
                               int cache_len, float sm_scale, ScoreWorkspace ws,
                               hipStream_t stream) {
  if (cache_len <= 0 || n_seq * n_head <= 0) return hipSuccess;
  dim3 grid(ws.n_chunk, n_seq * n_head);
  if (dtype == 0) {
    if (d == 128)
      hipLaunchKernelGGL((score_logits_f32_kernel<128>), grid, dim3(kThreads), 0, stream, (const float*)q, q_unit_stride,
                         rows, n_win, (const float*)k.ptr, k.seq_stride, k.head_stride, n_head, cache_len, sm_scale, ws);
    else
      hipLaunchKernelGGL((score_logits_f32_kernel<64>), grid, dim3(kThreads), 0, stream, (const float*)q, q_unit_stride,
                         rows, n_win, (const float*)k.ptr, k.seq_stride, k.head_stride, n_head, cache_len, sm_scale, ws);
    return hipGetLastError();
  }
  if (d == 128)
    hipLaunchKernelGGL((score_logits_mfma_kernel<128>), grid, dim3(kThreads), 0, stream,
                       (const uint16_t*)q, q_unit_stride, rows, n_win, (const uint16_t*)k.ptr,
                       k.seq_stride, k.head_stride, n_head, cache_len, sm_scale, ws);
  else
    hipLaunchKernelGGL((score_logits_mfma_kernel<64>), grid, dim3(kThreads), 0, stream,
                       (const uint16_t*)q, q_unit_stride, rows, n_win, (const uint16_t*)k.ptr,
                       k.seq_stride, k.head_stride, n_head, cache_len, sm_scale, ws);
  return hipGetLastError();
}

hipError_t launch_score_finalize(int n_unit, int n_win, int cache_len, ScoreWorkspace ws,
                                 float* log_scores, long long score_unit_stride,
                                 hipStream_t stream) {
  if (cache_len <= 0 || n_unit <= 0) return hipSuccess;
  dim3 grid((cache_len + 255) / 256, n_unit);
  hipLaunchKernelGGL(score_finalize_kernel, grid, dim3(256), 0, stream, n_win, cache_len, ws,
                     log_scores, score_unit_stride);
  return hipGetLastError();
}

}  // namespace scalekv
