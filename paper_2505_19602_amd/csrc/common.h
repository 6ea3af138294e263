// Internal declarations shared by the ScaleKV HIP translation units (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace scalekv {

constexpr int kMaxWindow = 16;     // window rows held per unit by the score kernels
constexpr int kScoreChunk = 256;   // cached keys handled per workgroup in the score kernels
constexpr int kShortLen = 1536;    // longest cache that one workgroup ranks in LDS (rank.h)
constexpr int kLogitPad = 64;      // logits row stride is the cache length rounded up to this

// A cache viewed by kernels: base pointer plus strides in elements.
struct KvView {
  const void* ptr;
  long long seq_stride;
  long long head_stride;
};

struct WindowRows {
  int row[kMaxWindow];
};

struct ScoreWorkspace {
  float* logits;    // [U][len_pad][kMaxWindow]  (key-major: the 16 window logits of a key are 64 B)
  float* partial;   // [U][n_chunk][2][kMaxWindow]  (row max, row sum of exp(logit - max))
  int len_pad;
  int n_chunk;
  float* scores;    // [U][len_pad]  log-scores
  float* groups;    // [U][len_pad / 32][2][kMaxWindow]  as `partial`, of 32 keys; where the index list is written later
};

// Optional parts of the selection (Sec. 3.3): positions preserved whatever their score
// (the observation window) and average pooling of the scores along the cache axis.
struct SelectExtras {
  int n_forced;             // 0..kMaxWindow
  int forced[kMaxWindow];   // distinct positions in [0, cache_len)
  int pool_w;               // odd, 1 = no pooling
};

inline int round_up(int x, int m) { return (x + m - 1) / m * m; }

// Raises a kernel's dynamic-LDS limit, once per device: the attribute belongs to the current
// device's copy of the code, so a second GPU needs its own call.  `done` holds one bit per
// device (devices 64 and up are simply set every time); any number of host threads may race
// here, the call is idempotent.
inline hipError_t allow_dynamic_lds(const void* kernel, int bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
  if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess && bit) done.fetch_or(bit, std::memory_order_release);
  return e;
}

// ---- launchers (each enqueues on `stream` and returns hipGetLastError()) ----

hipError_t launch_score_logits(int dtype, int n_seq, int n_head, int d, const void* q,
                               long long q_unit_stride, WindowRows rows, int n_win, KvView k,
                               int cache_len, float sm_scale, ScoreWorkspace ws,
                               hipStream_t stream);
hipError_t launch_score_finalize(int n_unit, int n_win, int cache_len, ScoreWorkspace ws,
                                 float* log_scores, long long score_unit_stride,
                                 hipStream_t stream);
// `keep` counts the forced positions of `extras` (NULL: none, no pooling) as well.
hipError_t launch_select(int n_unit, const float* scores, long long score_unit_stride,
                         int cache_len, int keep, int32_t* idx, const SelectExtras* extras,
                         hipStream_t stream);
// The whole ranking step (bf16 only), by a workgroup per unit in one launch, or by several in three launches where
// rank_spreads(): the logits of the window rows against the unit's cached keys, the row normalisers and the log-scores
// (Eq. 5), and the selection.  Returns hipErrorNotSupported where score_select_fits() says no (and for fp32 or
// very long caches), and the caller takes the launches of the single stages, which fill the chip whatever the units.
// Of `ws` the logits are used, and where the ranking is spread the scores and, for statistics, the place of the indices.
// Ranked steps of 300 queries that keep a quarter, us, this ranking / the single stages (d 128; units x rows; 16 x 6400 and
// 60 x 12000 lie beyond the line):
//   16 x 600: 22.0 / 21.9   16 x 1600: 26.7 / 28.6   16 x 4096: 39.4 / 38.4   16 x 6400: 51.9 / 51.0   60 x 12000: 167 / 164
//   64 x 600: 34.2 / 33.1   64 x 1600: 44.4 / 43.4   64 x 4096: 71.9 / 70.2   64 x 6400: 99.5 / 97.6   64 x 12000: 172 / 168
//   128 x 1600: 62.3 / 61.8   128 x 4096: 115.5 / 114.5   128 x 6400: 168 / 168     256 x 600: 56.5 / 60.8   256 x 4096: 185 / 218
//   256 x 12000: 545 / 577    d 64: 60 x 1600: 34.2 / 34.2   60 x 4096: 53.1 / 50.0   128 x 4096: 76.7 / 75.7   256 x 12000: 290 / 331
// Up to 128 units the two are close, so that there the line decides little about time; it stays where it is because the
// single stages round the row normalisers by chunks of 256 keys: rows at the border of a selection may differ in the last
// bit of their score.
inline bool score_select_fits(int dtype, int d, int n_unit, int cache_len) {
  return dtype == 1 && (d == 64 || d == 128) && cache_len <= 12288 && (n_unit >= 64 || cache_len <= 4096);
}
// Whether the ranking of a unit is spread over workgroups (three launches instead of one, the same rows bit for bit),
// where score_select_fits().  `small`: the attention goes to the kernel for small work, which ranks up to kShortLen rows in
// its own launch, and prunes.  Whole steps that keep a quarter, us, a workgroup per unit / spread:
//   300 queries, d 128: 8 units x 600: 19.2 / 19.9   8 x 800: 21.8 / 20.3   8 x 1600: 32.8 / 23.0   8 x 4096: 59.3 / 31.0
//     32 x 800: 29.6 / 29.2   32 x 1600: 43.1 / 36.3   64 x 800: 37.8 / 34.9   64 x 1600: 52.5 / 44.8   64 x 10000: 226 / 147
//     96 x 1000: 45.4 / 44.8   96 x 1600: 60.4 / 57.0   96 x 4096: 112 / 100   128 x 1600: 61.9 / 63.5   128 x 4096: 116 / 117
//     128 x 6000: 174 / 163   192 x 6000: 236 / 251
//   d 64: 8 x 1000: 16.5 / 17.5   32 x 1000: 22.5 / 24.3   32 x 1600: 30.4 / 27.6   64 x 1600: 37.3 / 34.8   96 x 1600: 43.2 / 43.4
//     96 x 4096: 74.7 / 75.0   96 x 6000: 109 / 100
//   small, units, queries, rows, d 128: 16, 8, 600: 16.3 / 17.6   16, 8, 800: 19.0 / 18.8   16, 256, 900: 23.0 / 22.1
//     32, 100, 900: 21.7 / 21.9   32, 448, 900: 33.3 / 37.0   32, 80, 1200: 24.6 / 23.1   32, 448, 1200: 37.6 / 40.7 (the kernel
//     for small work has become faster since the line was drawn)   48, 80, 1200: 25.7 / 27.5   64, 64, 1536: 29.9 / 32.0
//     64, 64, 2000: 46.6 / 37.4   32, 256, 4096: 73.9 / 49.3   96, 20, 2000: 44.7 / 44.7   128, 16, 2000: 46.7 / 52.3
//     d 64: 8, 8, 1000: 15.4 / 18.2   16, 256, 1400: 20.9 / 19.6   24, 160, 1400: 20.4 / 20.6   32, 128, 1400: 20.7 / 21.4
//     64, 32, 3000: 38.9 / 36.1   96, 32, 3000: 41.6 / 45.3
inline bool rank_spreads(int d, int n_unit, int cache_len, bool small) {
  if (small && cache_len <= kShortLen)
    return d == 128 ? n_unit <= (cache_len >= 1000 ? 32 : 16) && cache_len >= 800 : n_unit <= 24 && cache_len >= 1300;
  if (small || n_unit <= 64) return n_unit <= 64 && cache_len >= (d == 128 ? 800 : 1300);
  return d == 128 ? n_unit <= (cache_len <= 4096 ? 96 : 128) && cache_len > kShortLen : n_unit <= 96 && cache_len > 4096;
}
// Where the ranking is spread, whether the kernel for small work leaves the pruning to it: its own copying workgroups come
// behind the n_wg attending ones, and wait for a round of their own where those (nearly) fill the compute units.
// us, pruned by the small kernel / before (n_wg, d 128): 32 units, 80 queries, 1200 rows (160)
// 23.6 / 25.3; 48, 40, 2000 (144) 33.8 / 33.0; 48, 64, 2000 (192) 36.4 / 34.8; 32, 100, 1200 (224) 29.6 / 26.2;
// 64, 64, 1536 (256) 30.0 / 29.9; 16, 256, 4096 (256) 40.8 / 37.2.
inline bool small_pruned_before(long long n_wg) { return n_wg > 160; }
// Whether selection and pruning share a launch behind launch_score_logits: a workgroup per unit, or several where there are
// fewer units than compute units.  Up to 256 units; more are not served in one round (fp32 steps, us, two launches / one:
// 32 units x 585 rows 69.7 / 64.5, 128 x 200 31.9 / 28.1, 256 x 1200 148 / 144, 300 x 1200 185 / 197).
inline bool select_prunes(int n_unit) { return n_unit <= 256; }
// The workgroups of a unit that do so: as many as the compute units take at once, and at least 64 rows to each.
inline int select_parts(int n_unit, int rows) {
  const int most = n_unit < 256 ? 256 / n_unit : 1, full = (rows + 63) / 64;
  return most < full ? most : full > 1 ? full : 1;
}
// With `prune` the same launch then also prunes (Sec. 3.3): source row idx[t] of k
// (keys) / prune->v_src (values) goes to row t of the destination caches, and the n_app rows of
// k_cur / v_cur ([U, n_app, d], NULL: none) are appended behind the keep rows.
struct PruneTarget {
  KvView v_src, k_dst, v_dst;
  const void* k_cur;
  const void* v_cur;
  int n_app;
};
hipError_t launch_score_select(int dtype, int n_seq, int n_head, int d, const void* q, long long q_unit_stride,
                               WindowRows rows, int n_win, KvView k, int cache_len, float sm_scale,
                               ScoreWorkspace ws, int keep, int32_t* idx, const SelectExtras* extras,
                               const PruneTarget* prune, bool small, hipStream_t stream);
// What follows launch_score_logits: log-scores, selection and, with `prune`, the pruning in the same launch as
// the selection.  hipErrorNotSupported beyond 12288 rows.  Up to 2048 rows the selection forms the log-scores itself: one
// workgroup takes 4 us per 1024 rows for it, as long as a launch of its own that spreads it over the chip.
hipError_t launch_select_prune(int dtype, int n_seq, int n_head, int d, int n_win, ScoreWorkspace ws, KvView k,
                               int cache_len, int keep, int32_t* idx, const SelectExtras* extras, const PruneTarget* prune,
                               hipStream_t stream);
// first n_sink and last keep - n_sink positions of every unit (n_sink <= keep <= cache_len)
hipError_t launch_positional(int n_unit, int cache_len, int n_sink, int keep, int32_t* idx,
                             hipStream_t stream);
// Eq. 2 for the n_rows (<= kMaxWindow) query rows whose logits sit in `ws`: per row the
// attention mass on keys [hist_len, len) and the sum of its top_k largest weights on keys
// [0, hist_len), written to terms[((unit * n_samp) + row0 + row) * 2 + {0, 1}]
hipError_t launch_asi_terms(int n_unit, ScoreWorkspace ws, int n_rows, int hist_len, int len,
                            int top_k, float* terms, int n_samp, int row0, hipStream_t stream);
// Eq. 2 for all n_samp query rows of q ([U, n_samp, d]) without a workspace of logits: bf16 and top_k up to
// 256, hipErrorNotSupported otherwise (or where ws_bytes does not hold the candidates, or where the sizes are
// such that the route through the logits is the faster one)
hipError_t launch_asi_stream(int dtype, int n_seq, int n_head, int d, const void* q, int n_samp, KvView k,
                             int hist_len, int len, int top_k, float sm_scale, void* ws, size_t ws_bytes,
                             float* terms, hipStream_t stream);
// Streaming costs 20-50 us whatever the sizes (lists, merge, one workgroup per part and pass of 32 rows); the route
// through the logits costs little where there are few keys, but reads and ranks 64 bytes a key and row anew for
// every row.  Measured, us, logits / streamed (units x keys, query rows; d 128, K' 64):
//   few rows in all:  4 x 1100, 16: 17 / 29     64 x 2000, 16: 39 / 48     16 x 3500, 64: 95 / 150    256 x 1100, 1: 31 / 34
//   many:             128 x 400, 8: 29 / 24     64 x 2000, 32: 74 / 77     256 x 1100, 16: 87 / 38
//   few, long keys:   64 x 3500, 8: 49 / 50     48 x 6300, 16: 64 / 52     16 x 10585, 32: 82 / 80    256 x 3500, 1: 78 / 62
inline bool asi_stream_pays(int n_unit, int len, int n_samp) {
  const long long keys = (long long)n_unit * len;
  const int rows = n_samp < 32 ? n_samp : 32;
  if ((n_unit < 256 ? n_unit : 256) * rows >= (n_unit >= 128 ? 1024 : 2048)) return true;
  return rows == 32 ? keys >= 160000 : rows >= 8 ? keys >= 220000 : keys >= 800000 && len >= 3000;
}
// out[0], out[1] = means of the two columns of terms [n][2]; out[2] = their product
hipError_t launch_asi_mean(const float* terms, long long n, float* out, hipStream_t stream);
// Rows of a cache that the pruning writes (of all units, K and V) are what the attention reads next: they are stored so
// that they may stay in the caches, unless that is more than the last-level cache (256 MB) holds; then they go past it.
// compact_kernel, which reads every source row once, still gains from what little stays at 1.5 times that size, the
// ranking kernels, which read the keys a second time when they copy, do not.
// Pruning and the attention of a step behind it, us, through / past the caches (256 units; written, queries):
//   compact_kernel    213 MB, 64: 120 / 124, 256: 154 / 166    288 MB, 64: 164 / 164, 256: 198 / 204, 1024: 533 / 543
//     384 MB, 64: 217 / 206, 256: 252 / 256, 1024: 645 / 648    425 MB, 64: 251 / 230, 256: 275 / 269, 1024: 669 / 666
//     603 MB, 64: 359 / 317, 256: 382 / 365, 1024: 868 / 861
//     (alone, with nothing that reads its rows, past the caches from 70 MB on: 213 MB 83.5 / 77.0, 749 MB 277 / 250)
//   ranking kernels   213 MB, 64: 155 / 152, 256: 188 / 191, 1024: 462 / 463    288 MB, 64: 203 / 201, 256: 232 / 227,
//     1024: 539 / 530    341 MB, 64: 247 / 227, 256: 270 / 259, 1024: 593 / 593    425 MB, 64: 318 / 274, 256: 342 / 307
//     (3244 of 6489 rows, 425 MB, 256: 399 / 384, 1024: 743 / 753)
enum class CacheWriter { kCompact, kRanking };
inline bool rows_go_past_caches(CacheWriter by, int n_unit, long long rows, int row_bytes) {
  const long long limit = by == CacheWriter::kCompact ? 400000000 : 256000000;
  return 2 * rows * n_unit * row_bytes > limit;
}
hipError_t launch_compact(int dtype, int n_seq, int n_head, int d, KvView k_src, KvView v_src,
                          const int32_t* idx, int keep, const void* k_cur, const void* v_cur,
                          int n_cur, KvView k_dst, KvView v_dst, hipStream_t stream);
hipError_t launch_attend(int dtype, int n_seq, int n_head, int d, const void* q, int n_q, KvView k,
                         KvView v, int kv_len, float sm_scale, void* out, hipStream_t stream);
// the fp32 part of launch_attend
hipError_t launch_attend_f32(int n_unit, int n_head, int d, const void* q, int n_q, KvView k, KvView v,
                             int kv_len, float sm_scale, void* out, hipStream_t stream);

// bf16 attention for small work, with the pruning and, for short caches, the ranking in the same
// launch (step_small.hip).
struct SmallStep {
  int n_unit, n_head, d;
  const void* q;            // [U, n_q, d]
  int n_q;
  int tile_rows;            // query rows per workgroup, from small_tile_rows()
  void* out;                // [U, n_q, d]
  // keys: len1 rows of the source cache (rows idx[t], or row t), then len2 rows of k_cur / v_cur
  KvView k, v;
  const void *k_cur, *v_cur;
  int len1, len2;
  const int32_t* idx;       // [U, len1]; NULL: the first len1 rows
  KvView k_dst, v_dst;      // ptr NULL: no cache is written
  bool copy_kept;           // the len1 rows are written as well, not only the len2 behind them
  float sm_scale;
  // cache_len > 0 (at most kShortLen): rank the cache_len rows of k with the window queries and keep len1
  // of them (0 < len1 < cache_len); idx is not used, idx_out (may be NULL) receives the rows
  int cache_len;
  WindowRows rows;
  int n_win;
  int32_t* idx_out;
};
hipError_t launch_step_small(const SmallStep& s, hipStream_t stream);
// What a call of that kernel does besides the attention.
enum class SmallWork {
  kAttend,   // nothing
  kAppend,   // the map's rows are copied behind the cached ones
  kKeepAll,  // every cached row is copied as well
  kRanked,   // the kept rows, chosen in this launch, are copied
  kRankedBefore  // the kept rows, chosen in the launch before, are copied
};
// The same of a step that keeps `keep` of cache_len rows.
inline SmallWork step_work(int keep, int cache_len) {
  if (keep > 0 && keep < cache_len) return cache_len <= kShortLen ? SmallWork::kRanked : SmallWork::kRankedBefore;
  return keep > 0 ? SmallWork::kKeepAll : SmallWork::kAppend;
}
// Query rows per workgroup of that kernel for n_q bf16 queries over kv keys, 0 where the other kernels
// are the better ones.  A workgroup of it fills a compute unit, and its time grows with the rows it
// carries, so: the fewest rows with which the chip's 256 compute units take the launch in one round.
// Measured against ranking + pruning + pipelined attention (us, d 128; units, queries, cached, kept; this kernel's
// time stands first, also where the rule takes the other side; every row kept: see below):
//   16 rows:   16 x 144, 340, 80: 15.1 / 24.0       16 x 256, 1200, 300: 24.5 / 31.0
//   32 rows:   32 x 256, 380, 82: 20.0 / 26.0       8 x 1024, 1500, 700: 38.5 / 45.2
//   64 rows:   64 x 256, 380, 82: 24.7 / 27.0       16 x 1024, 400, 80: 35.3 / 36.0
//              16 x 576, 1200, 300, ranked before: 35.4 / 34.6  (the narrowest; head_dim 64, 16 x 1024, 820, 390: 30.0 / 34.2)
//   128 rows:  256 x 128, 300, 60: 25.4 / 27.6      (up to 320 keys)
//              128 x 256, 380, 82: 30.3 / 30.4      (longer: not worth it)
// From 64 rows on it is what the launch does besides the attention that pays: the attention alone is then faster in the
// pipelined kernel (64 x 144 queries, 300 keys: 12.1 / 10.2; 128 x 144, 300 keys, 128 rows: 17.9 / 10.4), and with few
// keys from 32 rows on (8 x 700, 64 keys: 7.1 / 5.3; 130: 8.0 / 7.9; 400: 10.3 / 11.7).  A ranking in the same launch
// is repeated by every workgroup of a unit: 64 rows pay up to 16 of those, 32 only with head_dim 64 (8 x 2048, 380, 82:
// 50.1 / 47.8, head_dim 64 33.5 / 35.2).  Without one 64 rows pay while
// the workgroups leave some compute units to those that copy, which otherwise wait for a round of their
// own (ranked before, 2500 cached, 300 kept: 64 x 144 44.8 / 45.0; 64 x 256 49.1 / 46.0; 16 x 1024 51.2 / 45.4), 128 rows do
// not.
// Appending alone copies least and gains least: head_dim 64, up to 224 workgroups (64 rows: 56 x 200, 500 keys: 11.5 / 12.5;
// 64 x 256, 256 workgroups: 16.2 / 12.3; thousands of keys: 224 x 62, 4035: 42.1 / 39.1); head_dim 128: 64 x 144, 500: 17.3 / 16.3.
// More units than compute units: two rounds are paid, which only maps of up to 16 queries stand
// (320 x 4, 65, 65: 8.1 / 10.1;  512 x 16, 69, 14: 18.1 / 18.4).
//
// keep_all_is_pipelined(): where every row is kept, the pipelined kernel copies the tiles that pass through it, while
// this one has workgroups for that behind the n_wg attending ones, of `rows` query rows, which read everything once
// more.  The pipelined kernel has n_pipe workgroups, of 128 rows, each of which walks all keys: where they are few it loses by
// the length of the cache what it gains by copying.  Small / pipelined, us (units, queries, cached rows):
//   64 rows, d 128: 8, 1000, 800 (n_wg 128): 24.8 / 31.9   24, 465, 69 (168): 16.0 / 16.3   40, 200, 200 (160): 14.0 / 14.5
//     64, 144, 800 (192): 27.6 / 23.0   32, 400, 3000 (224): 64.3 / 55.9
//     d 64: 8, 1000, 800: 16.2 / 21.5   24, 500, 800 (192): 17.2 / 17.7   96, 103, 438 (192): 14.9 / 11.8   16, 900, 800 (240): 24.3 / 21.4
//     up to 223 workgroups with few keys, n_pipe 120: 20, 650, 101 (220): 12.6 / 13.5   24, 525, 26 (216): 11.0 / 12.2   (more keys:
//     40, 265, 1201 (200): 22.1 / 19.5; n_pipe 200: 200, 40, 200: 12.2 / 9.5)
//   32 rows, d 128 (n_wg, n_pipe): 16, 485, 230 (256, 64): 16.4 / 17.5   16, 485, 4009: 54.0 / 72.4   32, 254, 300 (256, 64):
//     16.0 / 15.5   32, 254, 1700: 36.9 / 39.0   32, 254, 4473: 67.6 / 85.6   60, 108, 550 (240, 60): 22.1 / 19.5   60, 108, 1700: 39.7 / 43.9
//     12, 546, 800 (216, 60): 17.4 / 26.1   32, 200, 800 (224, 64): 19.7 / 23.2   48, 100, 800 (192, 48): 19.6 / 24.0
//     40, 173, 221 (240, 80): 15.2 / 13.7   48, 160, 800 (240, 96): 24.9 / 21.8   128, 60, 800 (256, 128): 34.2 / 26.2
//     few keys, no wave of this kernel has a second chunk (ONE in step_small.hip): 48, 160, 70: 9.5 / 12.1
//     96, 60, 150: 9.7 / 11.1   128, 60, 150: 11.2 / 11.1
//     d 64: 64, 100, 800: 15.4 / 15.6   96, 60, 300: 10.9 / 9.7   96, 37, 1812: 24.6 / 26.9   120, 52, 4951: 73.8 / 61.6
//     128, 60, 800: 20.3 / 17.2   128, 60, 150: 7.0 / 8.5
//   16 rows, a pipelined workgroup to a unit.  Little work is done sooner in this kernel; how little depends on the idle
//   compute units, which it sends to copy.  d 128: 96, 30, 800: 23.0 / 24.9   128, 10, 800: 25.3 / 25.6   128, 10, 3000: 82.7 / 71.1
//     160, 10, 400: 20.4 / 18.0   192, 10, 200: 12.9 / 12.7   256, 4, 100: 7.7 / 9.2   256, 4, 140: 13.5 / 10.6   300, 10, 65: 8.2 / 10.2
//     300, 10, 100: 11.1 / 10.2   512, 4, 30: 8.9 / 8.7   512, 4, 100: 15.9 / 12.2   256, 10, 800: 50.0 / 35.8
//     d 64: 128, 10, 900: 15.2 / 19.2   144, 10, 900: 18.2 / 18.5   168, 10, 800: 19.4 / 17.0   192, 10, 400: 12.1 / 11.0   224, 10, 400:
//     12.9 / 11.9   256, 10, 800: 26.5 / 20.2   300, 4, 200: 8.9 / 10.4   384, 10, 200: 10.0 / 10.7
//   A new cache (keys and values, 4 bytes an element) beyond the last-level cache of 256 MB is written to the HBM while the
//   source is read from it.  This kernel keeps all compute units at that; the pipelined one those that have a unit, in the
//   last round too: taken where five eighths of the units' rounds over the chip are filled or more (at that line either is up
//   to 7 % the faster, by the cache's length).  8 queries, d 128:
//   128, 5000: 136.7 / 167.1   160, 3400: 120.6 / 129.6   160, 4200: 163.3 / 148.6   168, 3148: 119.5 / 124.7   168, 4200: 179.8 / 150.6
//     208, 4200: 237 / 179   256, 3000: 188 / 164   272, 3000: 195 / 218   288, 3000: 202 / 224   320, 2000: 162.1 / 161.2
//     320, 3000: 225 / 235   336, 3000: 240.5 / 239.0   384, 3000: 277 / 251      within: 288, 1500: 99.0 / 81.3
//     d 64: 272, 5000: 158 / 173      within: 160, 6000: 103.4 / 79.3
inline bool keep_all_is_pipelined(int d, int n_unit, int n_q, int rows, long long n_wg, int kv) {
  const long long n_pipe = (long long)n_unit * ((n_q + 127) / 128);  // pipelined workgroups
  if (rows >= 64) return d == 128 ? n_wg > 128 : n_wg > 192 && (n_wg >= 224 || n_pipe > 128 || kv >= 1024);
  if (rows == 32 && n_pipe >= (d == 128 ? 96 : 112)) return kv > 256;
  if (rows == 32) return kv > 256 && kv <= 1280 && (n_unit >= 96 || (d == 128 && n_unit >= 32 && n_wg > 224));
  const long long elements = (long long)n_unit * kv * d;  // of the new keys, and as many values
  if (4 * elements > (256 << 20)) {
    const int rounds = (n_unit + 255) / 256;
    return 16 * n_unit >= 10 * 256 * rounds;
  }
  const bool idle = (d == 64 ? n_unit : n_wg) < 192;
  return n_unit >= 128 && elements >= (idle ? 8000000 : d == 64 ? 5000000 : n_unit >= 384 ? 2000000 : 3850000);
}
inline int small_tile_rows(int dtype, int d, int n_unit, int n_q, int kv, SmallWork work) {
  if (dtype != 1) return 0;
  constexpr int kComputeUnits = 256;
  int rows = 16;
  long long n_wg = 0;
  for (; rows <= 128; rows *= 2)
    if ((n_wg = (long long)n_unit * ((n_q + rows - 1) / rows)) <= kComputeUnits) break;
  if (work == SmallWork::kKeepAll && keep_all_is_pipelined(d, n_unit, n_q, rows > 128 ? 16 : rows, n_wg, kv)) return 0;
  if (rows > 128) return n_q <= 16 ? 16 : 0;
  if (rows == 32 && work == SmallWork::kAttend && kv <= 128) return 0;
  if (rows <= 32) return rows;
  if (rows == 128) return work == SmallWork::kRanked && kv <= 320 ? rows : 0;
  const bool spare = n_wg <= kComputeUnits * 7 / 8;
  const bool pays = (work == SmallWork::kRanked && (d == 64 || n_q <= 1024)) ||
                    (work == SmallWork::kRankedBefore && spare) || work == SmallWork::kKeepAll ||
                    (work == SmallWork::kAppend && d == 64 && spare);
  return pays ? rows : 0;
}

// Forms of the pipelined attention kernel.
enum class PipeForm {
  kPlain,  // 128 query rows and four waves per workgroup, two (head_dim 64: three) workgroups per compute unit
  kWide,   // 256 query rows and eight waves, one workgroup per compute unit: half the tile transfers
  kSplit   // 128 query rows, two (three) groups of four waves that share them and split the keys
};
// Measured (us; units x queries, keys; d 128 unless stated):
//   split / plain, up to a workgroup per compute unit (a plain one leaves half of it idle):
//     16 x 1024, 400: 12.5 / 13.3   1200: 22.3 / 27.4   4000: 59 / 79      64 x 400, 1200: 23.5 / 28.2
//     few keys do not pay for the join: 16 x 1024, 130: 9.1 / 8.8   64 keys: 7.4 / 6.1
//     more workgroups than compute units: 48 x 700, 1200: 45 / 35
//     d 64: 64 x 400, 400: 9.7 / 10.1   1200: 16.1 / 20.4   4000: 38.6 / 58.4   130: 7.5 / 6.7
//   wide / plain, from a workgroup per compute unit on: 256 x 4096, 3000: 1425 / 1469     256 x 129, 3000: 92 / 98
//     few keys do not pay (start and end of a workgroup have no neighbour to hide behind): 256 x 4096, 1200: 646 / 647
//     300: 261 / 234
//     a last round that is nearly empty, or rows of padding, cost twice as much:
//     256 x 320, 3000: 169 / 161    512 x 576, 3000: 520 / 475     64 x 2304, 3000: 241 / 223
//     less than a round: 96 x 320, 3000: 77 / 75
inline PipeForm pipe_form(int d, int n_unit, int n_q, int kv) {
  constexpr int kComputeUnits = 256;
  const long long wide = (long long)n_unit * ((n_q + 255) / 256), plain = (long long)n_unit * ((n_q + 127) / 128);
  if (plain <= kComputeUnits) return kv >= 320 ? PipeForm::kSplit : PipeForm::kPlain;
  if (d != 128 || wide < kComputeUnits || kv < 2048) return PipeForm::kPlain;
  // rounds over the chip, in hundredths; a plain round that is at most half full takes 70
  const long long rest = plain % (2 * kComputeUnits);
  const long long wide_rounds = (wide + kComputeUnits - 1) / kComputeUnits * 100;
  const long long plain_rounds = plain / (2 * kComputeUnits) * 100 + (rest == 0 ? 0 : rest <= kComputeUnits ? 70 : 100);
  return wide_rounds * 96 <= plain_rounds * 100 ? PipeForm::kWide : PipeForm::kPlain;
}
inline int pipe_rows(PipeForm form) { return form == PipeForm::kWide ? 256 : 128; }  // query rows per workgroup

// Whether a step that keeps all `cached` rows leaves their copy to that kernel.  In its wide form the copies of both segments
// pass through the loop, where the map's own rows cost more than at its end: with few cached rows beside 4096 of the map
// a copy before it is as good or better.  Steps, us, copied before / by the kernel: 256 units x 4096 queries, 100 rows
// 1973 / 1993, 800 2296 / 2311, 1500 2623 / 2628, 2500 3087 / 3089, 6489 4990 / 4870.  With fewer queries the line lies
// too high, by up to 3 % of a step: 256 x 2304, 200 728 / 720, 1000 942 / 924, 1500 1085 / 1060; 128 x 2040, 300 298 / 292.
inline bool pipe_copies_cache(int d, int n_unit, int n_q, int cached) {
  return pipe_form(d, n_unit, n_q, cached + n_q) != PipeForm::kWide || 2LL * cached >= n_q;
}

// bf16: the pipelined kernel used when there is enough work for it.  Keys and values are the
// first len1 rows of the caches k, v followed by the len2 rows of the dense tensors k2, v2
// ([U, len2, d]; may be NULL when len2 == 0).  With `copy` the kernel also copies the second segment into rows
// [len1, len1 + len2) of the caches named there, which are k and v, or (`both`) both segments from row 0 on, and the caches
// are others than those it reads; they must have room for the rows.  `start` / `stop`
// (either may be NULL): events that receive the kernel's own start and end times; they ride on
// the kernel's dispatch, so unlike hipEventRecord they put no operation of their own on the stream.
struct AttendCopy {
  KvView k, v;
  bool both;
};
hipError_t launch_attend_pipe(int n_unit, int n_head, int d, const void* q, int n_q, KvView k, KvView v,
                              int len1, const void* k2, const void* v2, int len2, const AttendCopy* copy,
                              float sm_scale, void* out, hipStream_t stream,
                              hipEvent_t start = nullptr, hipEvent_t stop = nullptr);

// ---- device helpers ----
// Workgroup coordinates as the kernels read them.  A build with SCALEKV_REVERSE_WG
// (python -m paper_2505_19602_amd.build --variant reversed_order) walks every grid backwards:
// workgroup i does the work that workgroup n-1-i does in the plain build.  No result may depend
// on which workgroup runs first; a test compares the two builds bit for bit.
#if defined(SCALEKV_REVERSE_WG)
#define SCALEKV_WG_X ((int)(gridDim.x - 1 - blockIdx.x))
#define SCALEKV_WG_Y ((int)(gridDim.y - 1 - blockIdx.y))
#define SCALEKV_WG_Z ((int)(gridDim.z - 1 - blockIdx.z))
#else
#define SCALEKV_WG_X ((int)blockIdx.x)
#define SCALEKV_WG_Y ((int)blockIdx.y)
#define SCALEKV_WG_Z ((int)blockIdx.z)
#endif
// Consecutive workgroup ids go round-robin over the eight XCDs, each with an L2 of its own.  This
// renumbers them so that the ids an XCD receives are consecutive (the tail, fewer than eight, keeps
// its ids): workgroups that read the same rows then share an L2.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_order(int wg, int n_wg) {
  const int per = n_wg / kXcds;
  return wg < per * kXcds ? wg % kXcds * per + wg / kXcds : wg;
}
// Butterflies over the four rows of 16 lanes of a wave: lanes l and l^16, then l and l^32, in
// registers.  The swap hands every lane {own value, partner's value} in some order; maximum and
// sum do not care which is which.
__device__ __forceinline__ void swap16(float x, float& a, float& b) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap32(float x, float& a, float& b) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
// x of lane 16 ROW + l % 16, in every lane.
template <int ROW>
__device__ __forceinline__ float from_row(float x) {
  float lo, hi;
  swap32(x, lo, hi);  // the lower half in both halves, the upper half in both
  const float half = ROW / 2 ? hi : lo;
  swap16(half, lo, hi);
  return ROW % 2 ? hi : lo;
}
__device__ __forceinline__ float xor16_max(float x) { float a, b; swap16(x, a, b); return fmaxf(a, b); }
__device__ __forceinline__ float xor32_max(float x) { float a, b; swap32(x, a, b); return fmaxf(a, b); }
__device__ __forceinline__ float xor16_sum(float x) { float a, b; swap16(x, a, b); return a + b; }
__device__ __forceinline__ float xor32_sum(float x) { float a, b; swap32(x, a, b); return a + b; }

// The number of log2 units a row maximum may grow before the running offset is moved and the accumulators are
// rescaled.
constexpr float kRescaleThreshold = 8.f;
// Running maximum of rows that have met no key yet, in kernels that take the weight of a logit s as
// exp2(s * scale_log2e - maximum * scale_log2e): finite, and finite when it has been scaled, so that keys
// whose logits are all -inf add weights of zero and not NaN.  (The 2^-20 by which it stays below FLT_MAX
// covers the rounding of the division and of the product.)
inline float no_maximum(float scale_log2e) { return -0x1.fffff0p127f / (scale_log2e > 1.f ? scale_log2e : 1.f); }

// ---- shared between the score finalisation and the fused select ----
// Row normalisers max_j + log Z_j of the window rows from the per-chunk (max, sum exp) pairs, into
// row_shift[kMaxWindow] (LDS; 0 from n_win on), by the whole workgroup (at least 2 kMaxWindow threads).
// The pairs of up to kStatChunks chunks come into LDS (stage) at once: a thread that walks them in
// global memory pays a latency per chunk (14 us at 26 chunks).  A barrier at the end.
constexpr int kStatChunks = 64;
__device__ __forceinline__ void score_row_shifts(const ScoreWorkspace& ws, int unit, int n_win,
                                                 float (&stage)[kStatChunks * 2 * kMaxWindow],
                                                 float (&row_shift)[kMaxWindow]) {
  const float* part = ws.partial + (long long)unit * ws.n_chunk * 2 * kMaxWindow;
  const int tid = threadIdx.x, j = tid;
  float m = -INFINITY;
  const bool staged = ws.n_chunk <= kStatChunks;
  if (staged) {
    for (int e = tid; e < ws.n_chunk * 2 * kMaxWindow; e += blockDim.x) stage[e] = part[e];
    __syncthreads();
  }
  if (tid < kMaxWindow) {
    float z = 0.f;
    if (staged) {
#pragma unroll 4
      for (int c = 0; c < ws.n_chunk; ++c) m = fmaxf(m, stage[c * 2 * kMaxWindow + j]);
#pragma unroll 4
      for (int c = 0; c < ws.n_chunk; ++c)
        z += stage[c * 2 * kMaxWindow + kMaxWindow + j] * expf(stage[c * 2 * kMaxWindow + j] - m);
    } else {
      for (int c = 0; c < ws.n_chunk; ++c) m = fmaxf(m, part[c * 2 * kMaxWindow + j]);
      for (int c = 0; c < ws.n_chunk; ++c)
        z += part[c * 2 * kMaxWindow + kMaxWindow + j] * expf(part[c * 2 * kMaxWindow + j] - m);
    }
    row_shift[j] = j < n_win ? m + logf(z) : 0.f;
  }
  __syncthreads();
}
// log s_i = logsumexp_j(logit[i][j] - shift_j) from the n_win logits of one key
template <typename Shift>
__device__ __forceinline__ float log_sum_rows(float (&la)[kMaxWindow], int n_win, const Shift& row_shift) {
  float top = -INFINITY;
#pragma unroll
  for (int j = 0; j < kMaxWindow; ++j) {
    la[j] = j < n_win ? la[j] - row_shift[j] : -INFINITY;
    top = fmaxf(top, la[j]);
  }
  float acc = 0.f;
#pragma unroll
  for (int j = 0; j < kMaxWindow; ++j) acc += j < n_win ? expf(la[j] - top) : 0.f;
  return top + logf(acc);
}
// the same for one key of the workspace; row_shift lives in LDS
__device__ __forceinline__ float score_log_sum(const ScoreWorkspace& ws, int unit, int key, int n_win,
                                               const float* row_shift) {
  const float* lg = ws.logits + ((long long)unit * ws.len_pad + key) * kMaxWindow;
  float la[kMaxWindow];
#pragma unroll
  for (int j4 = 0; j4 < kMaxWindow; j4 += 4) {
    const float4 x = *(const float4*)(lg + j4);
    la[j4] = x.x; la[j4 + 1] = x.y; la[j4 + 2] = x.z; la[j4 + 3] = x.w;
  }
  return log_sum_rows(la, n_win, row_shift);
}

}  // namespace scalekv
