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

constexpr int kThreads = kScoreChunk;  // bf16 kernel: 64 keys per wave

// fp32 logits kernel, plain FMA in channel order.  16 waves per 256-key chunk: wave w takes keys
// 64 (w % 4) .. +63, one per lane, and window rows 4 (w / 4) .. +3, so that a chunk has four times
// the waves of a thread-per-key form and a row costs a thread 4 instead of 16 fma per channel.
// The chunk's keys come through LDS, 32 channels at a time, as whole 128-byte pieces (a thread
// walking its own row in global memory touches 64 lines per instruction); the next piece is
// requested before this one is used.  LDS rows are 36 floats apart: an odd number of 16-byte
// units, no bank conflicts.  The window queries are wave-uniform and arrive as scalars.  Bound by
// latency at the sizes in use: 585 keys x 32 units (96 workgroups), 22 us thread-per-key.
template <int D>
__global__ __launch_bounds__(1024) void score_logits_f32_kernel(
    const float* __restrict__ q, long long q_unit_stride, WindowRows rows, int n_win,
    const float* __restrict__ k, long long k_seq_stride, long long k_head_stride, int n_head,
    int cache_len, float sm_scale, ScoreWorkspace ws) {
  constexpr int kPiece = 32, kStride = kPiece + 4, kRows = 4;
  __shared__ __attribute__((aligned(16))) float ks[kScoreChunk * kStride];
  __shared__ float red_max[kScoreChunk / 64][kMaxWindow];
  __shared__ float red_sum[kScoreChunk / 64][kMaxWindow];

  const int unit = SCALEKV_WG_Y;
  const int seq = unit / n_head, head = unit - seq * n_head;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = wave & 3, row0 = kRows * (wave >> 2);
  const int key0 = SCALEKV_WG_X * kScoreChunk;
  const float* ku = k + seq * k_seq_stride + head * k_head_stride;
  const float* qr[kRows];
#pragma unroll
  for (int j = 0; j < kRows; ++j) {
    int row = 0;
#pragma unroll
    for (int t = 0; t < kMaxWindow; ++t) row = t == row0 + j ? rows.row[t] : row;  // (an index would put rows into LDS)
    qr[j] = q + unit * q_unit_stride + (long long)row * D;
  }

  static_assert(kScoreChunk * kPiece / 4 == 2 * 1024, "two 16-byte vectors per thread and piece");
  constexpr int kPer = kPiece / 4;
  const int ld_key = tid / kPer, ld_c = 4 * (tid % kPer);  // and the same 128 keys on
  const float* ld_a = ku + (long long)min(key0 + ld_key, cache_len - 1) * D + ld_c;  // clamp: legal address, value unused
  const float* ld_b = ku + (long long)min(key0 + ld_key + 128, cache_len - 1) * D + ld_c;
  float4 stage_a = *(const float4*)ld_a, stage_b = *(const float4*)ld_b;
  float acc[kRows] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int c0 = 0; c0 < D; c0 += kPiece) {
    __syncthreads();  // the previous piece has been used
    *(float4*)(ks + ld_key * kStride + ld_c) = stage_a;
    *(float4*)(ks + (ld_key + 128) * kStride + ld_c) = stage_b;
    __syncthreads();
    if (c0 + kPiece < D) {
      stage_a = *(const float4*)(ld_a + c0 + kPiece);
      stage_b = *(const float4*)(ld_b + c0 + kPiece);
    }
    const float* krow = ks + (64 * group + lane) * kStride;
#pragma unroll
    for (int c = 0; c < kPiece; c += 4) {
      const float4 kv = *(const float4*)(krow + c);
#pragma unroll
      for (int j = 0; j < kRows; ++j) {
        acc[j] = fmaf(qr[j][c0 + c], kv.x, acc[j]);
        acc[j] = fmaf(qr[j][c0 + c + 1], kv.y, acc[j]);
        acc[j] = fmaf(qr[j][c0 + c + 2], kv.z, acc[j]);
        acc[j] = fmaf(qr[j][c0 + c + 3], kv.w, acc[j]);
      }
    }
  }

  const int key = key0 + 64 * group + lane;
  const bool valid = key < cache_len;
#pragma unroll
  for (int j = 0; j < kRows; ++j) acc[j] *= sm_scale;
  if (valid)
    *(float4*)(ws.logits + ((long long)unit * ws.len_pad + key) * kMaxWindow + row0) =
        make_float4(acc[0], acc[1], acc[2], acc[3]);
#pragma unroll
  for (int j = 0; j < kRows; ++j) {
    const float x = valid ? acc[j] : -INFINITY;
    float m = x;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    float e = valid ? expf(x - m) : 0.f;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off);
    if (lane == 0) { red_max[group][row0 + j] = m; red_sum[group][row0 + j] = e; }
  }
  __syncthreads();
  if (tid < kMaxWindow) {
    float m = -INFINITY;
    for (int w = 0; w < kScoreChunk / 64; ++w) m = fmaxf(m, red_max[w][tid]);
    float ssum = 0.f;
    for (int w = 0; w < kScoreChunk / 64; ++w)
      if (red_max[w][tid] > -INFINITY) ssum += red_sum[w][tid] * expf(red_max[w][tid] - m);
    float* part = ws.partial + ((long long)unit * ws.n_chunk + SCALEKV_WG_X) * 2 * kMaxWindow;
    part[tid] = m;
    part[kMaxWindow + tid] = ssum;
  }
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
  if (tid < kMaxWindow) {
    float mm = -INFINITY;
    for (int w = 0; w < kThreads / 64; ++w) mm = fmaxf(mm, red_max[w][tid]);
    float ssum = 0.f;
    for (int w = 0; w < kThreads / 64; ++w)
      if (red_max[w][tid] > -INFINITY) ssum += red_sum[w][tid] * expf(red_max[w][tid] - mm);
    float* part = ws.partial + ((long long)unit * ws.n_chunk + SCALEKV_WG_X) * 2 * kMaxWindow;
    part[tid] = mm;
    part[kMaxWindow + tid] = ssum;
  }
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
      hipLaunchKernelGGL((score_logits_f32_kernel<128>), grid, dim3(1024), 0, stream, (const float*)q, q_unit_stride,
                         rows, n_win, (const float*)k.ptr, k.seq_stride, k.head_stride, n_head, cache_len, sm_scale, ws);
    else
      hipLaunchKernelGGL((score_logits_f32_kernel<64>), grid, dim3(1024), 0, stream, (const float*)q, q_unit_stride,
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
