// Top-k of Sec. 3.3: a workgroup selects for one (sequence, head) unit.  Where it prunes as well, several may share a
// unit: each selects the same rows and copies a part of them.
//
// Scores are mapped to order-preserving unsigned keys; an 8-bit radix
// select of up to four passes finds the key T of the keep-th largest score; one stable pass then
// emits, in ascending index order, every index with key > T and the first
// (keep - #greater) indices with key == T.  Only integer compares are involved,
// so the result is deterministic and ties always go to the lower index.
//
// Two optional parts of the paper's selection are folded into the key set-up:
// average pooling of the scores along the cache axis (odd width, zeros beyond the
// ends; done on log-scores as a log-sum-exp, which ranks the same), and positions
// that are preserved whatever their score (the observation window): those take no part in
// the search, are emitted with the others, and `keep` counts them.
#include <type_traits>

#include "common.h"
#include "radix_select.h"
#include "rank.h"
#include "score_mfma.h"

namespace scalekv {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kLdsKeys = 12288;  // units up to this many scores keep their keys in LDS
static_assert(kLdsKeys == 12288 && kLdsKeys == 1024 * kLongMaxPer, "score_select_fits() in common.h states the same limit");

// What a kernel that ranks from the keys needs: bf16 storage only.
struct ScoreInputs {
  const uint16_t* q;        // [U, *, D]; window queries are rows `rows` of every unit
  long long q_unit_stride;
  WindowRows rows;
  const uint16_t* k;        // cache
  long long k_seq_stride, k_head_stride;
  int n_head;
  float sm_scale;
  // Pruning by the same workgroup (Sec. 3.3: the selected rows are preserved): after the
  // selection, row idx[t] of the source caches is copied to row t of the destination caches, and
  // n_app rows of k_cur / v_cur ([U, n_app, D]) are appended behind the kept ones.  Off if
  // k_dst == NULL.  v_src may differ from the key cache in base and strides; strides in elements.
  const uint16_t* v_src;
  long long v_seq_stride, v_head_stride;
  uint16_t* k_dst;
  uint16_t* v_dst;
  long long kd_seq_stride, kd_head_stride, vd_seq_stride, vd_head_stride;
  const uint16_t* k_cur;
  const uint16_t* v_cur;
  int n_app;
  bool past_caches;         // rows_go_past_caches()
};

// Pruning of one unit by one workgroup, or by `parts` of them: the kept rows (and, if asked, the map's rows behind them)
// into the destination.
// vec_log2: 16-byte vectors per row.
template <int THREADS>
__device__ __forceinline__ void prune_unit(const ScoreInputs& si, int unit, int keep, const int32_t* list, int vec_log2,
                                           int part = 0, int parts = 1) {
  typedef unsigned int vec4 __attribute__((ext_vector_type(4)));
  constexpr int kFly = 4;          // vectors in flight per thread and tensor
  const int tid = threadIdx.x;
  const int seq = unit / si.n_head, head = unit - seq * si.n_head;
  const vec4* ksrc = (const vec4*)(si.k + seq * si.k_seq_stride + head * si.k_head_stride);
  const vec4* vsrc = (const vec4*)(si.v_src + seq * si.v_seq_stride + head * si.v_head_stride);
  vec4* kdst = (vec4*)(si.k_dst + seq * si.kd_seq_stride + head * si.kd_head_stride);
  vec4* vdst = (vec4*)(si.v_dst + seq * si.vd_seq_stride + head * si.vd_head_stride);
  const vec4* kcur = (const vec4*)si.k_cur + ((long long)unit * si.n_app << vec_log2);
  const vec4* vcur = (const vec4*)si.v_cur + ((long long)unit * si.n_app << vec_log2);
  const int share = (keep + si.n_app + parts - 1) / parts << vec_log2;
  const int first = part * share, total = min((keep + si.n_app) << vec_log2, first + share);
  // (the attention reads the kept rows next: plain stores, which may leave them in the caches, unless they are too many.
  // 256 units, 246 of 546 rows, 576 queries, the whole step: 110.8 us with streaming stores, 107.2 so.  Two loops: of
  // two kinds of store in one the compiler makes plain ones.)
  auto copy = [&](auto past) __attribute__((always_inline)) {
#pragma unroll 1
    for (int f0 = first + tid; f0 < total; f0 += THREADS * kFly) {
      vec4 a[kFly], b[kFly];
#pragma unroll
      for (int u = 0; u < kFly; ++u) {
        // (lanes past the end re-read the last vector and store nothing: a branch around the loads
        // costs the kernel 30 registers)
        const int f = min(f0 + u * THREADS, total - 1);
        const int row = f >> vec_log2, c = f & ((1 << vec_log2) - 1);
        const bool kept = row < keep;
        const long long o = ((long long)(kept ? list[row] : row - keep) << vec_log2) + c;
        a[u] = __builtin_nontemporal_load((kept ? ksrc : kcur) + o);
        b[u] = __builtin_nontemporal_load((kept ? vsrc : vcur) + o);
      }
#pragma unroll
      for (int u = 0; u < kFly; ++u) {
        const int f = f0 + u * THREADS;
        if (f >= total) continue;
        if constexpr (decltype(past)::value) {
          __builtin_nontemporal_store(a[u], kdst + f);
          __builtin_nontemporal_store(b[u], vdst + f);
        } else {
          kdst[f] = a[u];
          vdst[f] = b[u];
        }
      }
    }
  };
  if (si.past_caches) copy(std::true_type{});
  else copy(std::false_type{});
}

// Units too long for their keys to stay in LDS: scores given, keys formed anew in each pass.
__global__ __launch_bounds__(kThreads) void select_far_kernel(const float* __restrict__ scores, long long score_unit_stride,
                                                              int cache_len, int keep, int32_t* __restrict__ idx,
                                                              SelectExtras ex) {
  __shared__ __attribute__((aligned(16))) uint32_t hist[kRadixHistWords];
  __shared__ uint32_t wave_gt[kWaves], wave_eq[kWaves];
  const int unit = SCALEKV_WG_X;
  const int tid = threadIdx.x;
  const float* s = scores + unit * score_unit_stride;
  const int pool_r = (ex.pool_w - 1) / 2;
  auto key_at = [&](int i) -> uint32_t {
    for (int j = 0; j < ex.n_forced; ++j)
      if (ex.forced[j] == i) return 0xffffffffu;
    if (pool_r > 0) return order_key(pooled_log([&](int t) { return s[t]; }, i, cache_len, pool_r));
    return order_key(s[i]);
  };

  // ---- radix select: T = key of the keep-th largest ----
  uint32_t T, need_eq;  // need_eq: how many keys equal to T are taken (>= 1)
  radix_kth_largest<kThreads>(key_at, cache_len, (uint32_t)keep, hist, T, need_eq);

  // ---- stable emission ----
  const int per = (cache_len + kThreads - 1) / kThreads;
  const int lo = min(tid * per, cache_len), hi = min(lo + per, cache_len);
  uint32_t n_gt = 0, n_eq = 0;
  for (int i = lo; i < hi; ++i) {
    const uint32_t kk = key_at(i);
    n_gt += kk > T;
    n_eq += kk == T;
  }
  // exclusive block scan of (n_gt, n_eq)
  const int lane = tid & 63, wave = tid >> 6;
  const uint32_t sg = wave_prefix_sum(n_gt, lane), se = wave_prefix_sum(n_eq, lane);
  if (lane == 63) { wave_gt[wave] = sg; wave_eq[wave] = se; }
  __syncthreads();
  uint32_t base_g = 0, base_e = 0;
  for (int w = 0; w < wave; ++w) { base_g += wave_gt[w]; base_e += wave_eq[w]; }
  const uint32_t ex_g = base_g + sg - n_gt, ex_e = base_e + se - n_eq;
  uint32_t pos = ex_g + min(ex_e, need_eq);
  uint32_t eq_seen = ex_e;
  int32_t* out = idx + (long long)unit * keep;
  for (int i = lo; i < hi; ++i) {
    const uint32_t kk = key_at(i);
    if (kk > T) {
      out[pos++] = i;
    } else if (kk == T) {
      if (eq_seen < need_eq) out[pos++] = i;
      ++eq_seen;
    }
  }
}

// The whole ranking step of Sec. 3.3 and the pruning in one kernel, a workgroup per unit, for short caches
// (rank.h): nothing but the index list leaves the compute unit
// between the keys and the pruned rows.  EXTRAS: forced positions and pooling may be asked for.
// 256 units, 546 cached rows, 246 kept: 30.6 us with the logits through global memory, 26.3 here; 16-256 units,
// 70-400 rows: 13-17 -> 8-13 us.
template <int D, int THREADS, bool EXTRAS>
__global__ __launch_bounds__(THREADS) void rank_short_kernel(int cache_len, int keep, int32_t* __restrict__ idx,
                                                             int n_win, SelectExtras ex, ScoreInputs si) {
  extern __shared__ __attribute__((aligned(16))) float short_logits[];
  __shared__ RankShortLds lds;
  const int unit = SCALEKV_WG_X;
  const int seq = unit / si.n_head, head = unit - seq * si.n_head;
  rank_short<D, THREADS, EXTRAS>(si.q + unit * si.q_unit_stride, si.rows, n_win,
                                 si.k + seq * si.k_seq_stride + head * si.k_head_stride, cache_len, keep, si.sm_scale,
                                 ex, short_logits, lds, idx + (long long)unit * keep);
  if (si.k_dst != nullptr) prune_unit<THREADS>(si, unit, keep, lds.list, D == 128 ? 4 : 3);
}

// The same for longer ones.  256 units, 3350 cached rows, 1622 kept: 138 us, 148 with every logit through
// the workspace; 192 units, 2535 rows, ranking alone: 37 us against 46; 512 units, 2516 rows, 328 kept:
// a step of 144 queries 189 -> 174 us.
template <int D, int PER, bool EXTRAS>
__global__ __launch_bounds__(1024) void rank_long_kernel(int cache_len, int keep, int32_t* __restrict__ idx, int n_win,
                                                         SelectExtras ex, ScoreInputs si, ScoreWorkspace ws) {
  extern __shared__ __attribute__((aligned(16))) float long_turn[];
  __shared__ RankLongLds<PER> lds;
  const int unit = SCALEKV_WG_X;
  const int seq = unit / si.n_head, head = unit - seq * si.n_head;
  const int32_t* list = rank_long<D, PER, EXTRAS>(
      si.q + unit * si.q_unit_stride, si.rows, n_win, si.k + seq * si.k_seq_stride + head * si.k_head_stride, cache_len,
      keep, si.sm_scale, ex, long_turn, ws.logits + (long long)unit * ws.len_pad * kMaxWindow, lds,
      idx + (long long)unit * keep);
  if (si.k_dst != nullptr) prune_unit<1024>(si, unit, keep, list, D == 128 ? 4 : 3);
}

// ---- the ranking of a unit spread over workgroups, in three launches: logits, log-scores, selection and pruning.  Where
// there are few units, one workgroup to a unit leaves most of the chip idle: it forms the unit's logits, 16 exponentials
// twice for each key, and copies the kept rows, all through one compute unit.
// Normalisers and log-scores round as they do in rank_short (up to kShortLen rows) and rank_long: groups of 32 keys,
// merged in the order of those, so that the same rows are selected bit for bit.
// Bound by three launches and the chains in them: 16 units x 4096 rows, a quarter kept, d 128: 6.6 + 5.1 + 10.2 us, 47.7 by
// a workgroup per unit; 60 x 1733, d 64: 6.7 + 5.5 + 11.1, 26.0.  The log-scores formed by the workgroups that select, which
// saves a launch, is as fast up to 1000 rows and slower beyond (8 units x 2000 rows, whole step 27.4 / 29.5).
constexpr int kSpreadThreads = 256;
constexpr int kSpreadKeys = kSpreadThreads / 64 * 32;  // per workgroup of the first kernel

// Logits of 32 keys a wave, and their maximum and sum of exponentials for every window row.
template <int D>
__global__ __launch_bounds__(kSpreadThreads) void spread_logits_kernel(int cache_len, int n_win, ScoreInputs si,
                                                                       ScoreWorkspace ws) {
  const int unit = SCALEKV_WG_Y, lane = threadIdx.x & 63;
  const int group = SCALEKV_WG_X * (kSpreadThreads / 64) + (threadIdx.x >> 6);
  if (32 * group >= cache_len) return;
  const int seq = unit / si.n_head, head = unit - seq * si.n_head;
  score_bf16x8 qf[D / 32], kf[2][D / 32];
  score_load_keys<D, 2>(si.k + seq * si.k_seq_stride + head * si.k_head_stride, 32 * group, cache_len, kf);
  score_load_window<D>(si.q + unit * si.q_unit_stride, si.rows, n_win, qf);
  score_f32x4 c[2];
  float m, e;
  score_products<D, 2>(kf, qf, c);
  score_statistics<2>(c, 32 * group, cache_len, si.sm_scale, m, e);
  score_store_logits<2, true>(c, 32 * group, cache_len, ws.logits + (long long)unit * ws.len_pad * kMaxWindow, kMaxWindow);
  float* const stat = ws.groups + (long long)unit * ws.len_pad + group * (2 * kMaxWindow);
  if (lane < 2 * kMaxWindow) stat[lane] = lane < kMaxWindow ? m : e;  // (every lane l holds those of row l % 16)
}

// Log-scores of kSpreadThreads keys.
__global__ __launch_bounds__(kSpreadThreads) void spread_scores_kernel(int cache_len, int n_win, ScoreWorkspace ws) {
  static_assert(kSpreadThreads == kVirtualWaves * kMaxWindow, "a thread merges the groups of a virtual wave and row");
  __shared__ float wave_max[kVirtualWaves][kMaxWindow], wave_sum[kVirtualWaves][kMaxWindow];
  const int unit = SCALEKV_WG_Y, tid = threadIdx.x, i = tid & 15, g = (tid & 63) >> 4, first = tid / kMaxWindow;
  const int key = SCALEKV_WG_X * kSpreadThreads + tid, n_group = (cache_len + 31) / 32;
  const float* const lg = ws.logits + ((long long)unit * ws.len_pad + min(key, cache_len - 1)) * kMaxWindow;
  float la[kMaxWindow];  // (requested in front of the statistics)
#pragma unroll
  for (int j4 = 0; j4 < kMaxWindow; j4 += 4) {
    const float4 x = *(const float4*)(lg + j4);
    la[j4] = x.x; la[j4 + 1] = x.y; la[j4 + 2] = x.z; la[j4 + 3] = x.w;
  }
  const float* const stat = ws.groups + (long long)unit * ws.len_pad + i;
  float m_run = -INFINITY, e_run = 0.f;
  if (first < n_group) {
    m_run = stat[first * (2 * kMaxWindow)];
    e_run = stat[first * (2 * kMaxWindow) + kMaxWindow];
  }
#pragma unroll 4
  for (int group = first + kVirtualWaves; group < n_group; group += kVirtualWaves)
    join_keys(m_run, e_run, stat[group * (2 * kMaxWindow)], stat[group * (2 * kMaxWindow) + kMaxWindow]);
  wave_max[first][i] = m_run;
  wave_sum[first][i] = e_run;
  __syncthreads();
  float vm[4], ve[4], shift[kMaxWindow];
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    vm[x] = wave_max[4 * g + x][i];
    ve[x] = wave_sum[4 * g + x][i];
  }
  const int turns = (min(n_group, kVirtualWaves) + 3) / 4;
  row_shifts(cache_len <= kShortLen ? row_shift<false>(vm, ve, turns) : row_shift<true>(vm, ve, turns), shift);
  const float score = log_sum_rows(la, n_win, shift);
  if (key < cache_len) ws.scores[(long long)unit * ws.len_pad + key] = score;
}

template <int D, int PER, bool EXTRAS>
hipError_t launch_long(int n_unit, int cache_len, int keep, int32_t* idx, int n_win, const SelectExtras& ex,
                       const ScoreInputs& si, ScoreWorkspace ws, hipStream_t stream) {
  static std::atomic<uint64_t> configured{0};  // LDS above 64 KB per workgroup has to be asked for
  const hipError_t e = allow_dynamic_lds((const void*)rank_long_kernel<D, PER, EXTRAS>, kLongTurnBytes, configured);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((rank_long_kernel<D, PER, EXTRAS>), dim3(n_unit), dim3(1024), kLongTurnBytes, stream, cache_len,
                     keep, idx, n_win, ex, si, ws);
  return hipGetLastError();
}

template <int D, int THREADS, bool EXTRAS>
hipError_t launch_short(int n_unit, int cache_len, int keep, int32_t* idx, int n_win, const SelectExtras& ex,
                        const ScoreInputs& si, hipStream_t stream) {
  static std::atomic<uint64_t> configured{0};  // LDS above 64 KB per workgroup has to be asked for
  const hipError_t e = allow_dynamic_lds((const void*)rank_short_kernel<D, THREADS, EXTRAS>,
                                         rank_short_logit_bytes(kShortLen), configured);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((rank_short_kernel<D, THREADS, EXTRAS>), dim3(n_unit), dim3(THREADS),
                     rank_short_logit_bytes(cache_len), stream, cache_len, keep, idx, n_win, ex, si);
  return hipGetLastError();
}

// Selection for units whose keys fit in LDS (PER rows per thread): from scores, or (FROM_LOGITS) from the logits and
// chunk statistics of the workspace, log-scores formed here; and, if si.k_dst is there, the pruning by the same launch.
// Every one of a unit's `parts` workgroups selects, the first writes the index list, and each copies its share
// of the rows.
template <int PER>
struct SelectLds {
  __attribute__((aligned(16))) uint32_t hist[4 * 256];
  uint32_t keys[PER * kThreads];
  uint32_t wave_max[kWaves], wave_min[kWaves];
  uint32_t count[PER * 2 * kWaves];  // as in RankShortLds
};
template <int PER, bool FROM_LOGITS, bool COPIES>
__global__ __launch_bounds__(kThreads) void select_lds_kernel(const float* __restrict__ scores, long long score_unit_stride,
                                                              int cache_len, int keep, int32_t* __restrict__ idx,
                                                              ScoreWorkspace ws, int n_win, SelectExtras ex, ScoreInputs si,
                                                              int vec_log2, int parts) {
  extern __shared__ __attribute__((aligned(16))) int32_t select_list[];  // [keep], where rows are copied
  __shared__ SelectLds<PER> lds;
  __shared__ float row_shift[kMaxWindow], stage[FROM_LOGITS ? kStatChunks * 2 * kMaxWindow : 1];
  const int wg = xcd_order(SCALEKV_WG_X, gridDim.x);  // (what the workgroups of a unit read meets in one L2)
  const int unit = wg / parts, part = wg - unit * parts, tid = threadIdx.x;
  lds.hist[tid] = 0;
  if constexpr (FROM_LOGITS) score_row_shifts(ws, unit, n_win, stage, row_shift);
  float own[PER];
#pragma unroll
  for (int c = 0; c < PER; ++c) {
    const int key = tid + c * kThreads;
    if (key < cache_len) {
      if constexpr (FROM_LOGITS) own[c] = score_log_sum(ws, unit, key, n_win, row_shift);
      else own[c] = scores[unit * score_unit_stride + key];
    }
  }
  if constexpr (COPIES)
    select_scores<kThreads, PER, true>(own, cache_len, keep, ex, lds, select_list,
                                       part == 0 ? idx + (long long)unit * keep : nullptr);
  else
    select_scores<kThreads, PER, true>(own, cache_len, keep, ex, lds, nullptr, idx + (long long)unit * keep);
  if constexpr (COPIES) prune_unit<kThreads>(si, unit, keep, select_list, vec_log2, part, parts);
}

template <bool FROM_LOGITS, bool COPIES>
hipError_t launch_select_lds(int n_unit, const float* scores, long long score_unit_stride, int cache_len, int keep,
                             int32_t* idx, ScoreWorkspace ws, int n_win, const SelectExtras& ex, const ScoreInputs& si,
                             int vec_log2, hipStream_t stream) {
  const int parts = COPIES ? select_parts(n_unit, keep + si.n_app) : 1;
#define SCALEKV_SELECT(PER)                                                                                              \
  do {                                                                                                                   \
    static std::atomic<uint64_t> configured{0}; /* LDS above 64 KB per workgroup has to be asked for */                  \
    const hipError_t e = !COPIES ? hipSuccess                                                                            \
                                 : allow_dynamic_lds((const void*)select_lds_kernel<PER, FROM_LOGITS, COPIES>,           \
                                                     PER * kThreads * 4, configured);                                    \
    if (e != hipSuccess) return e;                                                                                       \
    hipLaunchKernelGGL((select_lds_kernel<PER, FROM_LOGITS, COPIES>), dim3(n_unit * parts), dim3(kThreads),              \
                       COPIES ? keep * 4 : 0, stream, scores, score_unit_stride, cache_len, keep, idx, ws, n_win, ex,    \
                       si, vec_log2, parts);                                                                             \
  } while (0)
  if (cache_len <= kThreads) SCALEKV_SELECT(1);
  else if (cache_len <= 2 * kThreads) SCALEKV_SELECT(2);
  else if constexpr (!FROM_LOGITS) {
    if (cache_len <= 4 * kThreads) SCALEKV_SELECT(4);
    else if (cache_len <= 8 * kThreads) SCALEKV_SELECT(8);
    else SCALEKV_SELECT(kLdsKeys / kThreads);
  }
#undef SCALEKV_SELECT
  return hipGetLastError();
}

bool plain(const SelectExtras& ex) { return ex.n_forced == 0 && ex.pool_w == 1; }

// The part of ScoreInputs that says what is copied.  Rows are counted in elements of two bytes.
void set_prune(ScoreInputs& si, const PruneTarget& p, KvView k, int n_unit, int n_head, int keep, int row_bytes, int elem,
               CacheWriter by) {
  const int x = elem / 2;
  si.n_head = n_head;
  si.k = (const uint16_t*)k.ptr; si.k_seq_stride = k.seq_stride * x; si.k_head_stride = k.head_stride * x;
  si.v_src = (const uint16_t*)p.v_src.ptr;
  si.v_seq_stride = p.v_src.seq_stride * x; si.v_head_stride = p.v_src.head_stride * x;
  si.k_dst = (uint16_t*)const_cast<void*>(p.k_dst.ptr); si.v_dst = (uint16_t*)const_cast<void*>(p.v_dst.ptr);
  si.kd_seq_stride = p.k_dst.seq_stride * x; si.kd_head_stride = p.k_dst.head_stride * x;
  si.vd_seq_stride = p.v_dst.seq_stride * x; si.vd_head_stride = p.v_dst.head_stride * x;
  si.k_cur = (const uint16_t*)p.k_cur; si.v_cur = (const uint16_t*)p.v_cur;
  si.n_app = p.k_cur ? p.n_app : 0;
  si.past_caches = rows_go_past_caches(by, n_unit, keep + si.n_app, row_bytes);
}
int log2_of(int x) { return 31 - __builtin_clz(x); }
// Selection from ws.scores, and the pruning if `si` says so.
hipError_t select_from_scores(int n_unit, int cache_len, int keep, int32_t* idx, ScoreWorkspace ws, const SelectExtras& ex,
                              const ScoreInputs& si, int vec_log2, hipStream_t stream) {
  return si.k_dst ? launch_select_lds<false, true>(n_unit, ws.scores, ws.len_pad, cache_len, keep, idx, ws, 0, ex, si,
                                                   vec_log2, stream)
                  : launch_select_lds<false, false>(n_unit, ws.scores, ws.len_pad, cache_len, keep, idx, ws, 0, ex, si,
                                                    vec_log2, stream);
}

__global__ void iota_kernel(int32_t* __restrict__ idx, int keep, long long total) {
  const long long e = (long long)SCALEKV_WG_X * blockDim.x + threadIdx.x;
  if (e < total) idx[e] = (int32_t)(e % keep);
}

// Position-only retention (the sliding-window and sinks-plus-recent policies the paper
// compares against in Sec. 4.1): every unit keeps the first n_sink and the last
// keep - n_sink positions of its cache_len rows.
__global__ void positional_kernel(int32_t* __restrict__ idx, int keep, int n_sink, int cache_len,
                                  long long total) {
  const long long e = (long long)SCALEKV_WG_X * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int t = (int)(e % keep);
  idx[e] = t < n_sink ? t : cache_len - keep + t;
}

}  // namespace

hipError_t launch_positional(int n_unit, int cache_len, int n_sink, int keep, int32_t* idx,
                             hipStream_t stream) {
  if (n_unit <= 0 || keep <= 0) return hipSuccess;
  const long long total = (long long)n_unit * keep;
  hipLaunchKernelGGL(positional_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
                     stream, idx, keep, n_sink, cache_len, total);
  return hipGetLastError();
}

hipError_t launch_select(int n_unit, const float* scores, long long score_unit_stride,
                         int cache_len, int keep, int32_t* idx, const SelectExtras* extras,
                         hipStream_t stream) {
  SelectExtras ex{};
  ex.pool_w = 1;
  if (extras) ex = *extras;
  if (n_unit <= 0 || keep <= 0 || cache_len <= 0) return hipSuccess;
  if (keep >= cache_len) {  // keep everything: identity, no ranking needed
    const long long total = (long long)n_unit * keep;
    hipLaunchKernelGGL(iota_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream,
                       idx, keep, total);
    return hipGetLastError();
  }
  if (cache_len <= kLdsKeys)
    return launch_select_lds<false, false>(n_unit, scores, score_unit_stride, cache_len, keep, idx, ScoreWorkspace{}, 0, ex,
                                          ScoreInputs{}, 0, stream);
  hipLaunchKernelGGL(select_far_kernel, dim3(n_unit), dim3(kThreads), 0, stream, scores, score_unit_stride,
                     cache_len, keep, idx, ex);
  return hipGetLastError();
}

hipError_t launch_select_prune(int dtype, int n_seq, int n_head, int d, int n_win, ScoreWorkspace ws, KvView k,
                               int cache_len, int keep, int32_t* idx, const SelectExtras* extras, const PruneTarget* prune,
                               hipStream_t stream) {
  SelectExtras ex{};
  ex.pool_w = 1;
  if (extras) ex = *extras;
  const int n_unit = n_seq * n_head;
  if (cache_len > kLdsKeys) return hipErrorNotSupported;
  if (n_unit <= 0 || keep <= 0 || cache_len <= 0) return hipSuccess;
  const int elem = dtype == 0 ? 4 : 2, vec_log2 = log2_of(d * elem / 16);
  ScoreInputs si{};
  if (prune) set_prune(si, *prune, k, n_unit, n_head, keep, d * elem, elem, CacheWriter::kCompact);
  if (cache_len <= 2 * kThreads)
    return si.k_dst
        ? launch_select_lds<true, true>(n_unit, nullptr, 0, cache_len, keep, idx, ws, n_win, ex, si, vec_log2, stream)
        : launch_select_lds<true, false>(n_unit, nullptr, 0, cache_len, keep, idx, ws, n_win, ex, si, vec_log2, stream);
  const hipError_t e = launch_score_finalize(n_unit, n_win, cache_len, ws, ws.scores, ws.len_pad, stream);
  if (e != hipSuccess) return e;
  return select_from_scores(n_unit, cache_len, keep, idx, ws, ex, si, vec_log2, stream);
}

hipError_t launch_score_select(int dtype, int n_seq, int n_head, int d, const void* q, long long q_unit_stride,
                               WindowRows rows, int n_win, KvView k, int cache_len, float sm_scale,
                               ScoreWorkspace ws, int keep, int32_t* idx, const SelectExtras* extras,
                               const PruneTarget* prune, bool small, hipStream_t stream) {
  SelectExtras ex{};
  ex.pool_w = 1;
  if (extras) ex = *extras;
  const int n_unit = n_seq * n_head;
  if (!score_select_fits(dtype, d, n_unit, cache_len)) return hipErrorNotSupported;
  if (n_unit <= 0 || keep <= 0 || cache_len <= 0) return hipSuccess;
  ScoreInputs si{};
  si.q = (const uint16_t*)q; si.q_unit_stride = q_unit_stride; si.rows = rows;
  si.k = (const uint16_t*)k.ptr; si.k_seq_stride = k.seq_stride; si.k_head_stride = k.head_stride;
  si.n_head = n_head; si.sm_scale = sm_scale;
  constexpr int kComputeUnits = 256;  // MI355X
  if (rank_spreads(d, n_unit, cache_len, small)) {
    if (prune) set_prune(si, *prune, k, n_unit, n_head, keep, d * 2, 2, CacheWriter::kRanking);
    const dim3 logit_grid((cache_len + kSpreadKeys - 1) / kSpreadKeys, n_unit);
    if (d == 128)
      hipLaunchKernelGGL(spread_logits_kernel<128>, logit_grid, dim3(kSpreadThreads), 0, stream, cache_len, n_win, si, ws);
    else
      hipLaunchKernelGGL(spread_logits_kernel<64>, logit_grid, dim3(kSpreadThreads), 0, stream, cache_len, n_win, si, ws);
    hipLaunchKernelGGL(spread_scores_kernel, dim3((cache_len + kSpreadThreads - 1) / kSpreadThreads, n_unit),
                       dim3(kSpreadThreads), 0, stream, cache_len, n_win, ws);
    return select_from_scores(n_unit, cache_len, keep, idx, ws, ex, si, log2_of(d / 8), stream);
  }
  if (prune) set_prune(si, *prune, k, n_unit, n_head, keep, d * 2, 2, CacheWriter::kRanking);
  if (cache_len <= kShortLen) {
#define SCALEKV_SHORT(T)                                                                             \
  (d == 128 ? plain(ex) ? launch_short<128, T, false>(n_unit, cache_len, keep, idx, n_win, ex, si, stream) \
                    : launch_short<128, T, true>(n_unit, cache_len, keep, idx, n_win, ex, si, stream)  \
   : plain(ex) ? launch_short<64, T, false>(n_unit, cache_len, keep, idx, n_win, ex, si, stream)           \
           : launch_short<64, T, true>(n_unit, cache_len, keep, idx, n_win, ex, si, stream))
    // More units than compute units: 512 threads, of which two workgroups share a compute unit up to about 736 rows
    // (23 KB of LDS and 80 bytes a row of 160 KB), and which wait for fewer waves at each barrier beyond.
    // 1024 / 512 threads, us, ranking and pruning a fifth, d 128: 512 units x 500 rows 50.3 / 38.1, x 900 67.4 / 64.0,
    // x 1536 91.1 / 87.0; 320 x 760 56.5 / 52.8; 800 x 1300 141.3 / 134.4.
    return n_unit > kComputeUnits ? SCALEKV_SHORT(512) : SCALEKV_SHORT(1024);
#undef SCALEKV_SHORT
  }
#define SCALEKV_LONG(D, PER)                                                                           \
  (plain(ex) ? launch_long<D, PER, false>(n_unit, cache_len, keep, idx, n_win, ex, si, ws, stream)       \
         : launch_long<D, PER, true>(n_unit, cache_len, keep, idx, n_win, ex, si, ws, stream))
  if (cache_len <= kLongInRegisters) return d == 128 ? SCALEKV_LONG(128, 4) : SCALEKV_LONG(64, 4);
  return d == 128 ? SCALEKV_LONG(128, kLongMaxPer) : SCALEKV_LONG(64, kLongMaxPer);
#undef SCALEKV_LONG
}

}  // namespace scalekv
