// bf16 attention for small work: where the pipelined kernel (attend_pipe.hip, 128 query rows per
// workgroup) would leave most of the chip idle (small_tile_rows() in common.h).  The same launch
// prunes and appends the cache, and where the cache is short enough (rank.h) it also ranks it:
// a whole step in one kernel.
//
// A step of this size is bound by latency: the launch, a chain of dependent loads, barriers, and how
// many workgroups there are.  So the waves of a workgroup share 16 QB query rows (or several such
// blocks) and split the keys among them, 32 at a time; their partial results are joined in LDS at
// the end.  Kept rows are read where they are in the source cache, through the index list, not from
// the pruned copy.  Who writes the pruned copy:
//   MODE kRank   the workgroup has the index list in LDS and writes the rows that its waves read for
//                the attention anyway (each chunk of 32 keys by one of the unit's workgroups)
//   MODE kGiven  the kept rows are known before the launch (an index list, or all of them):
//                workgroups behind the attending ones copy, on compute units that would be idle
// Measured (16 units; a step of 16 queries over 69 cached rows, 14 kept; before: ranking kernel, then
// attention kernel): 19.1 -> 11.0 us a step; 9 queries, 967 of 6477 rows kept, 24 units: compaction and
// attention 53 -> 19 us; 256 units, maps of 16-64 queries: 25-29 -> 13-18 us.
// Keys through the stage as whole rows instead of as operands, a row per lane (L2 to one compute unit: 37 bytes a
// nanosecond so, 70-140 of whole rows): 16 units, 1024 queries, 312 of 773 rows 50.8 -> 47.0 us; 16, 3 queries, 2924 rows, all
// kept 33.2 -> 26.3; 40 x 56, 1218 rows, literal order 35.6 -> 32.6.  One chunk to a wave (ONE), whose fewer registers let two
// workgroups share a compute unit: 256 units, 4 queries, 65 rows 8.5 -> 6.3; 230, 12, 30 7.2 -> 5.4; 96, 10, 200 9.3 -> 8.2.
//
// Both products are formed transposed, on MFMA 16x16x32 (lane = 16g + i):
//   A (16 x 32): lane holds row i, k-indices 8g..8g+7     B (32 x 16): lane holds column i, same k-indices
//   C (16 x 16): lane holds column i, rows 4g + v, v = 0..3
//   S^T[key][query] = K Q^T: A = key rows, 16 bytes per lane
//   O^T[chan][query] += V^T P^T over 32 keys.  S^T of the two 16-key blocks leaves keys 4g + v and
//   16 + 4g + v in lane group g: taken in that order as k-indices 8g..8g+7 they are the B operand;
//   the A operand then is channel i of the same eight keys, which the transposing LDS load
//   (ds_read_b64_tr_b16) delivers from V rows staged in LDS, 32 of them per wave.
#include "common.h"
#include "rank.h"

namespace scalekv {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kChunk = 32;                    // keys per wave and iteration
constexpr int kCopyFly = 4;                   // 16-byte vectors per thread and tensor of a copying workgroup
enum Mode { kGiven = 0, kRank = 1 };

struct SmallArgs {
  const uint16_t* q;
  uint16_t* out;
  // keys: len1 rows of the source cache (rows idx[t], or row t if idx is NULL), then len2 rows of k2 / v2
  const uint16_t *k1, *v1, *k2, *v2;
  long long k1_seq, k1_head, v1_seq, v1_head;
  // destination cache (kd NULL: nothing is written): rows 0.. are the kept ones, len2 rows behind them
  uint16_t *kd, *vd;
  long long kd_seq, kd_head, vd_seq, vd_head;
  const int32_t* idx;   // kGiven: [U, len1] or NULL
  int32_t* idx_out;     // kRank: [U, len1] or NULL
  int n_q, len1, len2, n_head;
  int n_tile;           // workgroups per unit that attend
  int blocks_log2;      // query blocks (of 16 QB rows) per workgroup
  int n_attend;         // attending workgroups
  int n_copy;           // kGiven: copying workgroups per unit
  int copy_from;        // kGiven: first destination row that is written
  float scale_log2e;
  float no_maximum;     // where the running maxima start
  // kRank
  WindowRows rows;
  int n_win, cache_len;
  float sm_scale;
};

template <int D>
struct SmallLds {
  static constexpr int kRowStride = D * 2 + 32;  // bytes; consecutive rows start 8 banks apart (mod 64)
  static constexpr int kStage = kChunk * kRowStride;
  static constexpr int kPart = D / 16 * 64 * 16;  // one wave's 16 x D partial output, fp32
  static constexpr int kWave = kStage > kPart ? kStage : kPart;
  static constexpr int kBytes = kWaves * kWave;
};

// ONE: no wave has more than one chunk of keys.  It then takes the keys as operands: the way through the stage is only
// longer, and a kernel that ends within 5 us is sensitive to its own length (80 units, 3 queries, 40 rows: 4.9 us through
// the stage, 4.8 with a branch around it).
template <int D, int QB, int MODE, bool ONE>
__global__ __launch_bounds__(kThreads) void step_small_kernel(SmallArgs a) {
  constexpr int NSL = D / 32;          // k-slabs of the first product
  constexpr int NCB = D / 16;          // 16-channel blocks of the output
  constexpr int VPR = D / 8;           // 16-byte vectors per row
  constexpr int RPI = 64 / VPR;        // V rows per load instruction
  constexpr int NV = kChunk / RPI;     // V vectors per lane and chunk
  using L = SmallLds<D>;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  __shared__ float part_m[kWaves][QB][16], part_l[kWaves][QB][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = lane & 15, g = lane >> 4;
  const int len1 = a.len1, kv = a.len1 + a.len2;
  int wg = SCALEKV_WG_X;

  if constexpr (MODE == kGiven) {
    if (wg >= a.n_attend) {  // a copying workgroup: kThreads * kCopyFly vectors of K and of V
      wg -= a.n_attend;
      const int unit = wg / a.n_copy;
      const int seq = unit / a.n_head, head = unit - seq * a.n_head;
      const u32x4* ks = (const u32x4*)(a.k1 + seq * a.k1_seq + head * a.k1_head);
      const u32x4* vs = (const u32x4*)(a.v1 + seq * a.v1_seq + head * a.v1_head);
      const u32x4* kc = (const u32x4*)(a.k2 + (long long)unit * a.len2 * D);
      const u32x4* vc = (const u32x4*)(a.v2 + (long long)unit * a.len2 * D);
      u32x4* kd = (u32x4*)(a.kd + seq * a.kd_seq + head * a.kd_head);
      u32x4* vd = (u32x4*)(a.vd + seq * a.vd_seq + head * a.vd_head);
      const int32_t* list = a.idx ? a.idx + (long long)unit * len1 : nullptr;
      const int f0 = a.copy_from * VPR + (wg - unit * a.n_copy) * (kThreads * kCopyFly) + tid;
      u32x4 x[kCopyFly], y[kCopyFly];
#pragma unroll
      for (int u = 0; u < kCopyFly; ++u) {
        const int f = f0 + u * kThreads, row = f / VPR, c = f % VPR;
        if (row < len1) {
          const int o = (list ? list[row] : row) * VPR + c;
          x[u] = __builtin_nontemporal_load(ks + o);
          y[u] = __builtin_nontemporal_load(vs + o);
        } else if (row < kv) {
          const int o = (row - len1) * VPR + c;
          x[u] = __builtin_nontemporal_load(kc + o);
          y[u] = __builtin_nontemporal_load(vc + o);
        }
      }
#pragma unroll
      for (int u = 0; u < kCopyFly; ++u) {
        const int f = f0 + u * kThreads;
        if (f / VPR < kv) {
          __builtin_nontemporal_store(x[u], kd + f);
          __builtin_nontemporal_store(y[u], vd + f);
        }
      }
      return;
    }
  }

  wg = xcd_order(wg, a.n_attend);  // a unit's workgroups share an L2
  const int unit = wg / a.n_tile, tile = wg - unit * a.n_tile;
  const int seq = unit / a.n_head, head = unit - seq * a.n_head;
  const int n_block = 1 << a.blocks_log2;
  const int block = wave & (n_block - 1), split = wave >> a.blocks_log2, n_split = kWaves >> a.blocks_log2;
  const int q0 = (tile * n_block + block) * (16 * QB);
  const uint16_t* qu = a.q + (long long)unit * a.n_q * D;
  const uint16_t* k1 = a.k1 + seq * a.k1_seq + head * a.k1_head;
  const uint16_t* v1 = a.v1 + seq * a.v1_seq + head * a.v1_head;
  const uint16_t* k2 = a.k2 + (long long)unit * a.len2 * D;
  const uint16_t* v2 = a.v2 + (long long)unit * a.len2 * D;

  // query fragments: B operand of the first product; rows past the end repeat the last, nothing is stored for them
  bf16x8 qf[QB][NSL];
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    const uint16_t* row = qu + (long long)min(q0 + 16 * b + i, a.n_q - 1) * D + 8 * g;
#pragma unroll
    for (int sl = 0; sl < NSL; ++sl) qf[b][sl] = *(const bf16x8*)(row + 32 * sl);
  }

  const int32_t* list;
  if constexpr (MODE == kRank) {
    __shared__ RankShortLds rank;
    SelectExtras none;
    rank_short<D, kThreads, false>(qu, a.rows, a.n_win, k1, a.cache_len, len1, a.sm_scale, none,
                                   reinterpret_cast<float*>(smem), rank,
                                   a.idx_out && tile == 0 ? a.idx_out + (long long)unit * len1 : nullptr);
    list = rank.list;
  } else {
    list = a.idx ? a.idx + (long long)unit * len1 : nullptr;
  }

  // ---- one chunk: lane l (and l + 32) knows the row of key l, with the top bit set for the map's own
  auto row_of = [&](int chunk) -> int {
    const int t = min(chunk * kChunk + (lane & 31), kv - 1);
    if (t >= len1) return (int)((unsigned)(t - len1) | 0x80000000u);
    if constexpr (MODE == kRank) return list[t];
    else return list ? list[t] : t;
  };
  // (keys as values: RPI whole rows to an instruction.  Fetched as operands, a row per lane and 16 bytes of it, every lane
  // is a request of its own: a quarter of the rate.)
  u32x4 kr[NV], vr[NV];
  auto load_rows = [&](int rows, const uint16_t* cached, const uint16_t* own, u32x4 (&x)[NV]) {
#pragma unroll
    for (int p = 0; p < NV; ++p) {
      const int r = __shfl(rows, RPI * p + lane / VPR);
      x[p] = *(const u32x4*)((r < 0 ? own : cached) + (long long)(r & 0x7fffffff) * D + 8 * (lane % VPR));
    }
  };
  auto load_k = [&](int rows) { load_rows(rows, k1, k2, kr); };
  auto load_v = [&](int rows) { load_rows(rows, v1, v2, vr); };

  f32x4 o[QB][NCB];
  float m_run[QB], l_run[QB];
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    m_run[b] = a.no_maximum;
    l_run[b] = 0.f;
#pragma unroll
    for (int c = 0; c < NCB; ++c) o[b][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  unsigned char* const stage = smem + wave * L::kWave;
  const int n_chunk = (kv + kChunk - 1) / kChunk;
  int rows = 0;
  bf16x8 kf[2][NSL];
  if (split < n_chunk) {
    rows = row_of(split);
    if constexpr (ONE) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const int r = __shfl(rows, 16 * kb + i);
        const uint16_t* row = (r < 0 ? k2 : k1) + (long long)(r & 0x7fffffff) * D + 8 * g;
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl) kf[kb][sl] = *(const bf16x8*)(row + 32 * sl);
      }
    } else {
      load_k(rows);
    }
    load_v(rows);
    if (!ONE && split + n_split < n_chunk) rows = row_of(split + n_split);
  }
  for (int chunk = split; chunk < n_chunk; chunk += ONE ? n_chunk : n_split) {
    const bool more = !ONE && chunk + n_split < n_chunk;
    // through the wave's stage, the keys first: what a wave asks of the LDS is done in order
    auto to_stage = [&](const u32x4 (&x)[NV]) {
#pragma unroll
      for (int p = 0; p < NV; ++p)
        *(u32x4*)(stage + (RPI * p + lane / VPR) * L::kRowStride + 16 * (lane % VPR)) = x[p];
    };
    if constexpr (!ONE) {
      to_stage(kr);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl)
          kf[kb][sl] = *(const bf16x8*)(stage + (16 * kb + i) * L::kRowStride + 64 * sl + 16 * g);
    }
    to_stage(vr);
    if constexpr (MODE == kRank) {
      // this chunk's rows into the destination: one wave of one of the unit's workgroups
      if (block == 0 && chunk % a.n_tile == tile) {
        uint16_t* kd = a.kd + seq * a.kd_seq + head * a.kd_head;
        uint16_t* vd = a.vd + seq * a.vd_seq + head * a.vd_head;
#pragma unroll
        for (int p = 0; p < NV; ++p) {
          const int t = chunk * kChunk + RPI * p + lane / VPR;
          if (t < kv) {
            *(u32x4*)(kd + (long long)t * D + 8 * (lane % VPR)) = kr[p];
            *(u32x4*)(vd + (long long)t * D + 8 * (lane % VPR)) = vr[p];
          }
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (more) {  // the next chunk is on its way while this one's weights are formed
      load_k(rows);
      load_v(rows);
      if (chunk + 2 * n_split < n_chunk) rows = row_of(chunk + 2 * n_split);
    }
    __builtin_amdgcn_sched_barrier(0);
    f32x4 s[QB][2];
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        s[b][kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl)
          s[b][kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb][sl], qf[b][sl], s[b][kb], 0, 0, 0);
      }
    if ((chunk + 1) * kChunk > kv) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (chunk * kChunk + 16 * kb + 4 * g + v >= kv)
#pragma unroll
            for (int b = 0; b < QB; ++b) s[b][kb][v] = -INFINITY;
    }
    // the exponent offset of a row moves only when its maximum has grown by more than
    // kRescaleThreshold in log2 units: until then the weights stay below 2^8
    float mx[QB];
    bool grow = false;
#pragma unroll
    for (int b = 0; b < QB; ++b) {
      float m = s[b][0][0];
#pragma unroll
      for (int x = 1; x < 8; ++x) m = fmaxf(m, s[b][x / 4][x % 4]);
      mx[b] = xor32_max(xor16_max(m));
      grow |= (mx[b] - m_run[b]) * a.scale_log2e > kRescaleThreshold;
    }
    if (__builtin_amdgcn_ballot_w64(grow) != 0) {
#pragma unroll
      for (int b = 0; b < QB; ++b) {
        const float m_new = fmaxf(m_run[b], mx[b]);
        const float alpha = __builtin_amdgcn_exp2f((m_run[b] - m_new) * a.scale_log2e);
        m_run[b] = m_new;
        l_run[b] *= alpha;
#pragma unroll
        for (int c = 0; c < NCB; ++c)
#pragma unroll
          for (int v = 0; v < 4; ++v) o[b][c][v] *= alpha;
      }
    }
    bf16x8 pf[QB];
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int b = 0; b < QB; ++b) {
      const float off = m_run[b] * a.scale_log2e;
#pragma unroll
      for (int x = 0; x < 8; x += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[b][x / 4][x % 4], a.scale_log2e, -off));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(s[b][x / 4][x % 4 + 1], a.scale_log2e, -off));
        const bf16x2 pr = {(__bf16)p0, (__bf16)p1};
        pf[b][x] = pr[0];
        pf[b][x + 1] = pr[1];
        // the row sum adds the rounded weights, the very numbers the MFMA multiplies by
        l_run[b] = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, l_run[b], false);
      }
    }
#pragma unroll
    for (int c = 0; c < NCB; ++c) {
      const unsigned char* p = stage + (4 * g + (i >> 2)) * L::kRowStride + 32 * c + 8 * (i & 3);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) s16x4*)(p + 16 * L::kRowStride));
      const bf16x8 vt = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
      for (int b = 0; b < QB; ++b) o[b][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt, pf[b], o[b][c], 0, 0, 0);
    }
  }

  // ---- join the splits of each query block: a common offset, then the sum over the splits
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    l_run[b] = xor32_sum(xor16_sum(l_run[b]));
    if (g == 0) {
      part_m[wave][b][i] = m_run[b];
      part_l[wave][b][i] = l_run[b];
    }
  }
  __syncthreads();  // also: every wave has left its stage
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    float m = -INFINITY, l = 0.f;
    for (int w = 0; w < n_split; ++w) m = fmaxf(m, part_m[w * n_block + block][b][i]);
    for (int w = 0; w < n_split; ++w)
      l += part_l[w * n_block + block][b][i] *
           __builtin_amdgcn_exp2f((part_m[w * n_block + block][b][i] - m) * a.scale_log2e);
    const float f = __builtin_amdgcn_exp2f((m_run[b] - m) * a.scale_log2e) / l;  // 0 for a wave without keys
    if (b > 0) __syncthreads();  // the previous round has been read
    f32x4* const mine = reinterpret_cast<f32x4*>(stage);
#pragma unroll
    for (int c = 0; c < NCB; ++c) mine[c * 64 + lane] = o[b][c] * f;
    __syncthreads();
    // channel block c of query block `block`, summed by wave `split` (mod n_split) of that block
    const int row = q0 + 16 * b + i;
    for (int c = split; c < NCB; c += n_split) {
      f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int w = 0; w < n_split; ++w)
        sum += reinterpret_cast<const f32x4*>(smem + (w * n_block + block) * L::kWave)[c * 64 + lane];
      if (row < a.n_q) {
        const bf16x2 lo = {(__bf16)sum[0], (__bf16)sum[1]}, hi = {(__bf16)sum[2], (__bf16)sum[3]};
        uint2 pk;
        pk.x = __builtin_bit_cast(uint32_t, lo);
        pk.y = __builtin_bit_cast(uint32_t, hi);
        *(uint2*)(a.out + ((long long)unit * a.n_q + row) * D + 16 * c + 4 * g) = pk;
      }
    }
  }
}

template <int D, int QB, int MODE, bool ONE>
hipError_t launch(const SmallArgs& a, int n_wg, int lds, hipStream_t stream) {
  static std::atomic<uint64_t> configured{0};  // LDS above 64 KB per workgroup has to be asked for
  const hipError_t e = allow_dynamic_lds((const void*)step_small_kernel<D, QB, MODE, ONE>, 128 * 1024, configured);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((step_small_kernel<D, QB, MODE, ONE>), dim3(n_wg), dim3(kThreads), lds, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_step_small(const SmallStep& s, hipStream_t stream) {
  if (s.n_unit <= 0 || s.n_q <= 0) return hipSuccess;
  SmallArgs a{};
  a.q = (const uint16_t*)s.q;
  a.out = (uint16_t*)s.out;
  a.k1 = (const uint16_t*)s.k.ptr; a.k1_seq = s.k.seq_stride; a.k1_head = s.k.head_stride;
  a.v1 = (const uint16_t*)s.v.ptr; a.v1_seq = s.v.seq_stride; a.v1_head = s.v.head_stride;
  a.k2 = (const uint16_t*)s.k_cur; a.v2 = (const uint16_t*)s.v_cur;
  a.kd = (uint16_t*)const_cast<void*>(s.k_dst.ptr); a.kd_seq = s.k_dst.seq_stride; a.kd_head = s.k_dst.head_stride;
  a.vd = (uint16_t*)const_cast<void*>(s.v_dst.ptr); a.vd_seq = s.v_dst.seq_stride; a.vd_head = s.v_dst.head_stride;
  a.idx = s.idx; a.idx_out = s.idx_out;
  a.n_q = s.n_q; a.len1 = s.len1; a.len2 = s.len2; a.n_head = s.n_head;
  a.scale_log2e = s.sm_scale * 1.4426950408889634f;
  a.no_maximum = no_maximum(a.scale_log2e);
  a.rows = s.rows; a.n_win = s.n_win; a.cache_len = s.cache_len; a.sm_scale = s.sm_scale;
  // Rows per workgroup: 16 on all eight waves; from 32 on, waves of 32 rows (half the reads of K and V
  // per product), one, two or four such blocks to a workgroup.
  const int tile_rows = s.tile_rows;
  if (tile_rows != 16 && tile_rows != 32 && tile_rows != 64 && tile_rows != 128) return hipErrorInvalidValue;
  const int QB = tile_rows == 16 ? 1 : 2;
  a.blocks_log2 = tile_rows == 128 ? 2 : tile_rows == 64 ? 1 : 0;
  a.n_tile = (s.n_q + tile_rows - 1) / tile_rows;
  a.n_attend = s.n_unit * a.n_tile;
  int n_wg = a.n_attend;
  const int d = s.d;
  if (!s.cache_len && a.kd) {
    a.copy_from = s.copy_kept ? 0 : s.len1;
    const int total = (s.len1 + s.len2 - a.copy_from) * (d / 8);
    a.n_copy = (total + kThreads * kCopyFly - 1) / (kThreads * kCopyFly);
    n_wg += s.n_unit * a.n_copy;
  }
  int lds = d == 128 ? SmallLds<128>::kBytes : SmallLds<64>::kBytes;
  if (s.cache_len) lds = lds > rank_short_logit_bytes(s.cache_len) ? lds : rank_short_logit_bytes(s.cache_len);
  const bool one = (s.len1 + s.len2 + kChunk - 1) / kChunk <= kWaves >> a.blocks_log2;
#define SCALEKV_SMALL(D, Q)                                                                                     \
  (s.cache_len ? launch<D, Q, kRank, false>(a, n_wg, lds, stream)                                               \
   : one ? launch<D, Q, kGiven, true>(a, n_wg, lds, stream) : launch<D, Q, kGiven, false>(a, n_wg, lds, stream))
  if (d == 128) return QB == 2 ? SCALEKV_SMALL(128, 2) : SCALEKV_SMALL(128, 1);
  return QB == 2 ? SCALEKV_SMALL(64, 2) : SCALEKV_SMALL(64, 1);
#undef SCALEKV_SMALL
}

}  // namespace scalekv
