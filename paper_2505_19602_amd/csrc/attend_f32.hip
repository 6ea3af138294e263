// fp32 attention of the current token map over [retained cache ; current map] (Sec. 3.1 / 3.3),
// fp32 throughout, on the fp32 matrix instruction 16x16x4.
//
// Both products are formed transposed, so that a lane owns one query column:
//   S^T[key][query] = K Q^T,   O^T[chan][query] += V^T P^T
// MFMA 16x16x4 operand layout (lane = 16g + i):
//   A (16 x 4): lane holds row i, k-index g       B (4 x 16): lane holds column i, k-index g
//   C (16 x 16): lane holds column i, rows 4g + v, v = 0..3
// The order in which a contraction runs is free, and so is the channel that an output row stands
// for.  Both are chosen so that every operand comes from global memory as 16 bytes per lane and
// nothing passes through LDS:
//   K, Q   a lane's vector t is channels 16t + 4g .. +3 of its row; element e serves step (t, e)
//   P      S^T leaves key 4g + v in register v: already the B operand of step v
//   V      a lane's vector (v, t) is channels 64t + 4i .. +3 of key 4g + v; element c serves the
//          output block (t, c), whose row i is channel 64t + 4i + c
// so that a lane's results for fixed v are four consecutive channels.
//
// Bound by the matrix pipe (64 flop per clock and SIMD): 145 TFLOP/s is what the library's fp32
// matrix product reaches.  A wave owns 16 QB query rows and walks blocks of 16 keys; K of the next
// block is requested when the scores are formed, V when it has been used, about a thousand clocks
// ahead of use.  A map of a few hundred queries alone leaves most of the chip idle (400 queries x
// 32 units are 416 waves of 32 rows for 1024 SIMDs), so the waves of a workgroup share their query
// rows and split the keys; their partial results are joined in LDS at the end.
// Two waves per SIMD (no accumulation registers: with them the compiler copied hundreds of registers a block and kept
// one wave per SIMD) cover what is serial in a block: the softmax between the products and the joins.
// 400 queries x 517 keys x 32 units: 59 us with one wave, 53 now (64 TFLOP/s; 416 workgroups, one or two to a compute
// unit); 400 x 900 x 512 units: 1214 -> 904 us, 104 TFLOP/s; 200 x 1600 x 32: 74 -> 60.
#include <type_traits>

#include "common.h"

namespace scalekv {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kBlockKeys = 16;
constexpr int kMaxSplit = 4;  // waves of a workgroup
// Running maximum of a wave that has met no key yet: finite, so that a wave whose keys all have logits of -inf
// adds weights of zero and not NaN (the maximum is subtracted before the logits are scaled).
constexpr float kNoMaximum = -__FLT_MAX__;

template <int D, int QB>
__global__ __launch_bounds__(64 * kMaxSplit) __attribute__((amdgpu_waves_per_eu(2))) void attend_f32_kernel(
    const float* __restrict__ q, int n_q, const float* __restrict__ k, long long k_seq_stride,
    long long k_head_stride, const float* __restrict__ v, long long v_seq_stride,
    long long v_head_stride, int kv_len, int n_head, int n_tile, int n_split, float scale_log2e,
    float* __restrict__ out) {
  constexpr int NT = D / 16;  // channel vectors of a K or Q row per lane
  constexpr int NO = D / 64;  // 64-channel groups of the output
  __shared__ f32x4 part[kMaxSplit][4][64];
  __shared__ float part_m[kMaxSplit][QB][16], part_l[kMaxSplit][QB][16];

  const int wg = xcd_order(SCALEKV_WG_X, gridDim.x);  // the tiles of a unit share an L2
  const int unit = wg / n_tile, tile = wg - unit * n_tile;
  const int seq = unit / n_head, head = unit - seq * n_head;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;
  const int q0 = tile * (16 * QB);
  const float* qu = q + (long long)unit * n_q * D;
  const float* ku = k + seq * k_seq_stride + head * k_head_stride;
  const float* vu = v + seq * v_seq_stride + head * v_head_stride;

  f32x4 kf[NT], vf[4][NO];
  auto load_k = [&](int block) {
    const float* row = ku + (long long)min(block * kBlockKeys + i, kv_len - 1) * D + 4 * g;
#pragma unroll
    for (int t = 0; t < NT; ++t) kf[t] = *(const f32x4*)(row + 16 * t);
  };
  auto load_v = [&](int block) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* row = vu + (long long)min(block * kBlockKeys + 4 * g + r, kv_len - 1) * D + 4 * i;
#pragma unroll
      for (int t = 0; t < NO; ++t) vf[r][t] = *(const f32x4*)(row + 64 * t);
    }
  };
  f32x4 qf[QB][NT];
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    const float* row = qu + (long long)min(q0 + 16 * b + i, n_q - 1) * D + 4 * g;  // rows past the end: never stored
#pragma unroll
    for (int t = 0; t < NT; ++t) qf[b][t] = *(const f32x4*)(row + 16 * t);
  }
  // (behind the queries, so that the loop waits for the keys alone when it begins a block: with the queries the
  // younger ones it waited for the values as well, requested only just before)
  __builtin_amdgcn_sched_barrier(0);
  const int n_block = (kv_len + kBlockKeys - 1) / kBlockKeys;
  load_k(wave);
  __builtin_amdgcn_sched_barrier(0);
  load_v(wave);
  __builtin_amdgcn_sched_barrier(0);
  f32x4 o[QB][NO][4];
  float m_run[QB], l_run[QB];
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    m_run[b] = kNoMaximum;
    l_run[b] = 0.f;
#pragma unroll
    for (int t = 0; t < NO; ++t)
#pragma unroll
      for (int c = 0; c < 4; ++c) o[b][t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // `more`: whether a block follows, whose keys and values are requested as soon as the products have left their
  // registers.  The last block is a copy of its own: a condition at the requests would let the compiler assume that
  // they may not have been made, and wait for everything, and requests that nobody needs keep the join waiting (128
  // units x 33 queries x 60 keys, a block per wave: 9.4 us with them, 8.1 without; 32 x 400 x 300, 16 rows: 38.0, 34.8;
  // head_dim 64, many rounds: 6-10 %).  With 32 rows of head_dim 128, which are taken where there is much to do, one
  // body is the faster (256 x 1024 x 600 768 us, 822 with two; 512 x 400 x 600 630 / 670): there the last request takes
  // the last row again, and is dropped.
  constexpr bool kSameBody = D == 128 && QB == 2;
  auto walk = [&](int block, auto more) __attribute__((always_inline)) {
    f32x4 s[QB];
#pragma unroll
    for (int b = 0; b < QB; ++b) s[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int b = 0; b < QB; ++b)
          s[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][e], qf[b][t][e], s[b], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(more)::value) load_k(block + n_split);
    __builtin_amdgcn_sched_barrier(0);
    if ((!decltype(more)::value || kSameBody) && (block + 1) * kBlockKeys > kv_len) {  // (only the last block may be)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (block * kBlockKeys + 4 * g + r >= kv_len)
#pragma unroll
          for (int b = 0; b < QB; ++b) s[b][r] = -INFINITY;
    }
    // the exponent offset of a row moves only when its maximum has grown by more than
    // kRescaleThreshold in log2 units: until then the weights stay below 2^8
    float mx[QB];
    bool grow = false;
#pragma unroll
    for (int b = 0; b < QB; ++b) {
      float m = fmaxf(fmaxf(s[b][0], s[b][1]), fmaxf(s[b][2], s[b][3]));
      mx[b] = xor32_max(xor16_max(m));
      grow |= (mx[b] - m_run[b]) * scale_log2e > kRescaleThreshold;
    }
    if (__builtin_amdgcn_ballot_w64(grow) != 0) {
#pragma unroll
      for (int b = 0; b < QB; ++b) {
        const float m_new = fmaxf(m_run[b], mx[b]);
        const float alpha = __builtin_amdgcn_exp2f((m_run[b] - m_new) * scale_log2e);
        m_run[b] = m_new;
        l_run[b] *= alpha;
#pragma unroll
        for (int t = 0; t < NO; ++t)
#pragma unroll
          for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) o[b][t][c][r] *= alpha;
      }
    }
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[b][r] = __builtin_amdgcn_exp2f((s[b][r] - m_run[b]) * scale_log2e);
        l_run[b] += s[b][r];
      }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int t = 0; t < NO; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int b = 0; b < QB; ++b)
            o[b][t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][t][c], s[b][r], o[b][t][c], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(more)::value) load_v(block + n_split);
    __builtin_amdgcn_sched_barrier(0);
  };
  if constexpr (kSameBody) {
    for (int block = wave; block < n_block; block += n_split) walk(block, std::true_type{});
  } else {
    int block = wave;  // (every wave has one)
    for (; block + n_split < n_block; block += n_split) walk(block, std::true_type{});
    walk(block, std::false_type{});
  }

  // ---- join the waves' parts: common offset, then sums over the waves, 64 channels at a time
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    l_run[b] = xor32_sum(xor16_sum(l_run[b]));
    if (g == 0) {
      part_m[wave][b][i] = m_run[b];
      part_l[wave][b][i] = l_run[b];
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    float m = part_m[0][b][i];
    for (int w = 1; w < n_split; ++w) m = fmaxf(m, part_m[w][b][i]);
    float l = 0.f;
    for (int w = 0; w < n_split; ++w)
      l += part_l[w][b][i] * __builtin_amdgcn_exp2f((part_m[w][b][i] - m) * scale_log2e);
    const float f = __builtin_amdgcn_exp2f((m_run[b] - m) * scale_log2e) / l;  // 0 for a wave without keys
#pragma unroll
    for (int t = 0; t < NO; ++t) {
      if (n_split > 1) {
        __syncthreads();  // the previous round has been read
#pragma unroll
        for (int r = 0; r < 4; ++r)
          part[wave][r][lane] = f32x4{o[b][t][0][r], o[b][t][1][r], o[b][t][2][r], o[b][t][3][r]} * f;
        __syncthreads();
      }
      // register r of lane (g, i): channels 64t + 16g + 4r .. +3 of query i
      for (int r = wave; r < 4; r += n_split) {
        f32x4 sum;
        if (n_split > 1) {
          sum = part[0][r][lane];
          for (int w = 1; w < n_split; ++w) sum += part[w][r][lane];
        } else {
          sum = f32x4{o[b][t][0][0], o[b][t][1][0], o[b][t][2][0], o[b][t][3][0]};
#pragma unroll
          for (int x = 1; x < 4; ++x)
            if (r == x) sum = f32x4{o[b][t][0][x], o[b][t][1][x], o[b][t][2][x], o[b][t][3][x]};
          sum *= f;
        }
        const int row = q0 + 16 * b + i;
        if (row < n_q)
          *(f32x4*)(out + ((long long)unit * n_q + row) * D + 64 * t + 16 * g + 4 * r) = sum;
      }
    }
  }
}

template <int D, int QB>
hipError_t launch(int n_unit, int n_head, const float* q, int n_q, KvView k, KvView v, int kv_len,
                  float sm_scale, float* out, hipStream_t stream) {
  const int n_tile = (n_q + 16 * QB - 1) / (16 * QB);
  // A wave per SIMD of the compute unit, each with at least one block of keys.  (Eight waves were
  // 10-20 % slower at every size tried, two or one equal at best and up to 3 times slower.)
  const int n_block = (kv_len + kBlockKeys - 1) / kBlockKeys;
  const int split = n_block >= kMaxSplit ? kMaxSplit : n_block >= 2 ? 2 : 1;
  // A third workgroup of 16 rows per compute unit (head_dim 128) pays while the keys are few: over many the three walk
  // through more rows than the caches hold (with three / two, us: 100 units x 200 queries, 300 keys 49.5 / 52.4, 450
  // 70.7 / 71.2, 511 78.1 / 75.5, 800 117 / 105; 256 x 200, 300 108 / 120, 511 174 / 164).  LDS that nothing uses keeps
  // it out.
  const int lds = D == 128 && QB == 1 && kv_len >= 480 ? 40 * 1024 : 0;
  hipLaunchKernelGGL((attend_f32_kernel<D, QB>), dim3(n_tile * n_unit), dim3(64 * split), lds, stream, q, n_q,
                     (const float*)k.ptr, k.seq_stride, k.head_stride, (const float*)v.ptr, v.seq_stride,
                     v.head_stride, kv_len, n_head, n_tile, split, sm_scale * 1.4426950408889634f, out);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attend_f32(int n_unit, int n_head, int d, const void* q, int n_q, KvView k, KvView v,
                             int kv_len, float sm_scale, void* out, hipStream_t stream) {
  const float* qp = (const float*)q;
  float* op = (float*)out;
  // 32 query rows per wave halve the reads of K and V per flop; 16 rows make twice as many workgroups and fewer padded
  // rows, and their joins take half as long.  The launch takes as long as the compute unit that has most to do, m1
  // workgroups of 16 rows or m2 of 32.  Two of 32 rows share a compute unit, and one that is left alone in the last of a
  // few rounds costs as much as two: then 32 rows are taken where m2 is even (or 1) and m1 twice that.
  // 16 / 32 rows, us, d 128: m 2 / 1  120 keys 10.9 / 12.2, 160 13.2 / 14.3, 300 19.4 / 18.4, 1200 57.9 / 47.3
  //   4 / 2  120 keys 20.1 / 21.3, 300 35.4 / 34.9   6 / 3  300 keys 49.7 / 61.3, 1600 207 / 185   9 / 5  400 keys 90 / 104
  //   12 / 6  120 keys 53.0 / 56.4, 300 99.4 / 95.9   36 / 18  200 keys 208 / 221, 300 284 / 279, 600 477 / 451
  // d 64 (half the reads to save): 4 / 2  160 keys 11.8 / 13.2, 300 18.1 / 18.0, 1200 54.6 / 49.4   7 / 4  120 keys 16.1 /
  //   17.4, 800 64.9 / 65.4   8 / 4  300 keys 32.9 / 30.7   18 / 9  100 keys 0.98 of the time, 40 1.05   36 / 18  40 0.99
  constexpr int kComputeUnits = 256;
  const long long m1 = ((long long)((n_q + 15) / 16) * n_unit + kComputeUnits - 1) / kComputeUnits;
  const long long m2 = ((long long)((n_q + 31) / 32) * n_unit + kComputeUnits - 1) / kComputeUnits;
  const bool even = m1 == 2 * m2 && (m2 == 1 || m2 % 2 == 0);
  const bool wide = d == 128 ? m1 > 1 && m2 * 12 <= m1 * 7 && kv_len >= (m1 >= 18 || even ? 240 : 1000)
                             : m1 > 3 && m2 * 11 <= m1 * 6 &&
                                   kv_len >= (m1 >= 32 ? 0 : m1 >= 16 ? 100 : m1 > 4 ? 160 : 300);
  if (d == 128)
    return wide ? launch<128, 2>(n_unit, n_head, qp, n_q, k, v, kv_len, sm_scale, op, stream)
                : launch<128, 1>(n_unit, n_head, qp, n_q, k, v, kv_len, sm_scale, op, stream);
  return wide ? launch<64, 2>(n_unit, n_head, qp, n_q, k, v, kv_len, sm_scale, op, stream)
              : launch<64, 1>(n_unit, n_head, qp, n_q, k, v, kv_len, sm_scale, op, stream);
}

}  // namespace scalekv
