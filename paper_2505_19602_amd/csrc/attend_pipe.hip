// bf16 MFMA attention for large query counts: the kernel that
// carries almost all of the flops of the ScaleKV step (Sec. 3.1 / 3.3: the current
// token map attends, unmasked, over the retained cache followed by its own keys).
//
// Shape of the computation (transposed formulation):
//   S^T[key][query] = K Q^T          A = K rows from LDS,  B = Q held in registers
//   O^T[chan][query] += V^T P^T      A = V^T from LDS,     B = P^T straight from the
//                                    registers the first product left it in.
// so one lane owns one query column: the softmax statistics are per-lane scalars.
//
// MFMA 16x16x32 operand layout (lane = 16g + i):
//   A (16 x 32): lane holds row i, k-indices 8g..8g+7
//   B (32 x 16): lane holds column i, k-indices 8g..8g+7
//   C (16 x 16): lane holds column i, rows 4g..4g+3
// A wave's block is 32 keys x 32 queries: two key tiles times two query tiles of S^T.  MFMA row 4a + v of
// key tile t is fed key row 16(a & 1) + 8(a >> 1) + 4t + v of the block, so the registers of both key tiles of a
// query tile are, in lane group g, the eight keys from 16(g & 1) + 8(g >> 1) on: taken as k-indices 8g..8g+7 they
// are the B operand of the second product.  (This order of the keys lets the LDS swizzle below
// separate the rows that neighbouring lanes read.)
//
// Why 16x16x32 and not 32x32x16: the chip is power-limited under this kernel, and the smaller instruction does the
// same products for less energy (issue loop on registers, normal operands: 2.05 PFLOP/s, 1.76 with
// 32x32x16 on the same card).
//
// Schedule.  The unit of work is a block of 32 keys, 32 queries of a wave: kSlots MFMAs for S^T, as many for O^T, and
// 48 vector instructions of softmax between them.  A wave works on three blocks at once: beside the softmax of block b
// it issues the scores of block b + 1 and the weighted values of block b - 1, an MFMA, a request to the LDS and a
// step of the softmax in turn (`slots`), so that within a wave the vector and the matrix pipe run side by side; a
// second wave per SIMD (third, head_dim 64), from another workgroup, covers what is left of the latencies.  LDS
// operands are requested a product ahead of the MFMAs that take them, into registers which the product before has
// left.  Every slot is fenced: the compiler otherwise gathers the vector instructions behind the MFMAs (1-3 % slower,
// head_dim 64).  The loop runs two tiles a turn and leaves at one place: with a second exit in its middle the
// compiler spilled 45 registers.
// 4096 queries x 5718 keys x 256 units, d 128: 2800 us with 32x32x16 and the three phases of a block in sequence;
// 2655 so with 16x16x32; 2625 in this order (1.17 PFLOP/s).  1024 x 1180 x 64: 46.0 -> 42.5 us.
//
// Data movement.  K and V tiles (64 keys x 256 B) go from HBM/L2 straight into LDS
// (global_load_lds, 16 B per lane, no registers), row-major, with the 16-byte
// chunks of each row XOR-swizzled so that operand reads are free of bank conflicts.
// The V^T operand is read with the transposing LDS load (ds_read_b64_tr_b16):
// inside a group of 16 lanes, lane i supplies the address of 4 elements and
// receives element (i & 3) of the data addressed by lanes (i >> 2) + 4r, r = 0..3.
// Two stages per workgroup and tensor (wide form: four).  One barrier per tile (`turn`), in the middle of the second
// product of its first half: a wave has then read all of K tile t and of V tile t - 1, and has waited for its share of
// K tile t + 1 and V tile t, which may be read from there on, while K tile t + 2 and V tile t + 1 (t + 4 and t + 3)
// are requested.
//
// Three forms, chosen by pipe_form() in common.h, which holds their times.  Plain: four waves, 128 query rows, two
// workgroups per compute unit (head_dim 64: three).  Wide (d 128): eight waves, 256 rows, one workgroup per compute
// unit.  Its waves share the tiles, so the transfers into the LDS, which cost energy and issue slots (without any the
// plain form is 20 % faster), are halved, and they are requested three tiles ahead.  Split: where there is at most one
// plain workgroup per compute unit, two (three) groups of four waves take the tiles of the same 128 rows in turn, each
// with stages of its own, and join their accumulators through the LDS at the end.
//
// Softmax.  The exponent offset of a query row is taken from the row's maximum
// over the first tile and then left alone: every later probability is exp2 of
// (score - offset), whatever its size, and the row sum adds the bf16-rounded
// probabilities, the very numbers the MFMA multiplies by.  (The maximum over the tile's first block, followed by its
// second where that lies more than kRescaleThreshold higher in some row of the wave: the largest weights are then 1 or
// little larger, and what is exactly 1 is not rounded.  Root mean square error against fp64, output rounding and
// all, 256 units x 576 queries x 822 keys, peaked weights: 1.847e-3, with the first block alone 1.858e-3.  The first
// block's softmax has no MFMAs beside it then; 110.1 us, 109.9 with the first block alone.)
// No running maximum is
// formed (it costs a sixth of the vector instructions of a block).  This is exact as
// long as nothing overflows, and fp32 / bf16 carry 2^127: at the end of the pass a lane
// checks that its share of the row sum is below 2^120 (scores up to 83 natural units above the
// first tile's maximum; an infinite weight or a NaN is still in the sum then) and, since huge values could overflow
// them even so, that its accumulators are finite.  The split form, whose groups are joined relative to the largest
// of their offsets, has lower limits, 2^100 (69 units) and 2^125: the join scales a sum by no less than 2^-126 or drops
// what is then below 2^-24 of the row.
// If any lane of the workgroup finds a failure (forced by the tests), the workgroup
// discards its result and repeats the whole pass with the classical scheme: running
// maximum per block, offsets moved (and O, l rescaled) when some row maximum grew by
// more than kRescaleThreshold in log2 units.
//
// Workgroups of one (sequence, head) unit are numbered so that they land on the
// same XCD and share its L2 while they stream the same K/V.
//
// Two key segments.  The keys are the first len1 rows of a cache followed by len2
// rows of a dense tensor (the current map's own K/V); each segment is walked in tiles
// of its own, so at most one ragged tile per segment is masked.  When asked to, every
// workgroup also copies its share of the second segment behind the first in the cache
// (rows len1 .. len1+len2-1): the append of the pruning step, done here because this
// kernel is bound by the matrix pipe and leaves the HBM idle, while a separate copy
// kernel would be bound by the HBM and leave the matrix pipe idle.  Where every cached row is kept, the first segment is
// read from the source cache and both are copied, tile by tile from the LDS, to the destination (kCopyBoth): the cache is
// read once, and its copy costs little beside the products.  Steps, us, a copy before / this: 168 units x 529 queries x
// 4582 rows 403 / 332; 80 x 140 x 4458 124 / 87; 168 x 340 x 569 60.3 / 40.4; 120 x 182 x 153 22.5 / 13.8; 256 x 4096 x
// 6489 5437 / 5300; head_dim 64, 32 x 700 x 6000 84.5 / 69.1, 60 x 300 x 500 21.5 / 14.7.
#include <hip/hip_ext.h>

#include "common.h"

namespace scalekv {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int TN = 64;               // keys per staged tile (two blocks of 32)

// What depends on head_dim.  head_dim 64 halves the tiles and the accumulators, so that three
// workgroups share a compute unit instead of two; per block of 32 keys its 8 MFMA (256 clocks) and
// its softmax (16 fma, 16 exp2, 16 others: 260 clocks) are about equal, and the third wave per SIMD
// lets the two pipes overlap.  4096 queries x 4420 keys x 256 units: 1240 us with 32x32x16, 1160 now (1.02 PFLOP/s);
// 1215 x 1648 x 60: 47.0 -> 43.5 us.
// LDS rows are swizzled in 16-byte chunks so that operand reads are free of bank conflicts: chunk c of
// row r sits in slot c ^ k_flip(r) of a K row, c ^ v_flip(r) of a V row and c ^ q_flip(r) of a query row.  Rows
// of 256 bytes all start in the same bank, of rows of 128 bytes every second.  The sixteen lanes that read
// one chunk of sixteen K rows differ in row bits 0, 1, 3 and 4, the eight groups of lanes that read 32 bytes
// each of eight V rows in bits 0, 1 and 4.
template <int D, int WAVES, int SPLIT>
struct Shape {
  static constexpr int kThreads = 64 * WAVES * SPLIT;
  static constexpr int kRows = 32 * WAVES;                // query rows per workgroup
  static constexpr int kStages = WAVES == 8 ? 4 : 2;
  static constexpr int kRowBytes = D * 2;
  static constexpr int kTileBytes = TN * kRowBytes;       // 16 KB (d 128), 8 KB
  static constexpr int kSlabs = D / 32;                   // k-slabs of the first product
  static constexpr int kBlocks = D / 16;                  // 16-channel blocks of the output
  static constexpr int kChunks = D / 8;                   // 16-byte chunks per row
  static constexpr int kRowsPerOp = 64 / kChunks;         // rows that one transfer of a wave covers
  static constexpr int kWaveRows = TN / WAVES;            // rows of a tile that one wave transfers
  static constexpr int kOps = kWaveRows / kRowsPerOp;     // transfers for them
  static constexpr int kQOps = 32 / kRowsPerOp;           // transfers for a wave's query rows
  static constexpr int kWavesPerSimd = D == 128 ? 2 : 3;
  __device__ static constexpr int k_flip(int r) {
    const int high = (r >> 4 & 1) | (r >> 3 & 1) << 1;
    return D == 128 ? (r & 3) | high << 2 : (r >> 1 & 1) | high << 1;
  }
  __device__ static constexpr int v_flip(int r) {
    return D == 128 ? (r & 3) << 1 | (r >> 4 & 1) << 3 : (r >> 1 & 1) << 1 | (r >> 4 & 1) << 2;
  }
  __device__ static constexpr int q_flip(int r) { return D == 128 ? r & 15 : r >> 1 & 7; }
};
// Measurement-only builds (python -m paper_2505_19602_amd.build --variant ...; never the library
// the tests or the bench's headline load): each takes one ingredient out of the kernel so that
// its share of the running time can be read off a timing.  Their results are wrong on purpose.
//   SCALEKV_ABLATE_SOFTMAX    probabilities are the raw scores converted to bf16: no exp2, no
//                             row sums, no overflow watch
//   SCALEKV_ABLATE_TRANSFER   only the tiles that fill the stages once are fetched (two of each group, wide form:
//                             four); later tiles re-use them
//   SCALEKV_TIMELINE          every workgroup records when it started, when its first tile had
//                             arrived, when it left the tile loop and when it ended (results stay
//                             correct); scalekv_timeline_read() hands the records to the host
template <int D, int WAVES, int SPLIT>  // K stages then V stages, of every group
constexpr int kLdsBytes = 2 * SPLIT * Shape<D, WAVES, SPLIT>::kStages * Shape<D, WAVES, SPLIT>::kTileBytes;
#if defined(SCALEKV_TIMELINE)
constexpr int kTimelineMaxWg = 8192;
// four readings of the 100 MHz counter, the hardware id register, the shader clock counter at start and end
constexpr int kTimelineWords = 7;
__device__ unsigned long long g_timeline[kTimelineMaxWg * kTimelineWords];
#define SCALEKV_STAMP(name) const unsigned long long name = __builtin_amdgcn_s_memrealtime()
#else
#define SCALEKV_STAMP(name)
#endif
// A pass without maxima: the largest share of a row sum that it may end with and, where groups are added up, the largest
// accumulator.
template <int SPLIT>
constexpr float kRowSumLimit = SPLIT > 1 ? 0x1p100f : 0x1p120f;
constexpr float kSplitOutputLimit = 0x1p125f;

// One 16-byte-per-lane transfer from global memory straight into LDS: lane l's vector comes
// from base + voff + IMM and lands at LDS byte lds_addr + IMM + 16 l (the instruction's
// immediate offset applies to both addresses).  The request is written in
// assembly on purpose: the compiler, when it knows about a global->LDS transfer, waits for
// it before the next LDS read of the same array, which would serialise the transfer of tile
// t+1 with the consumption of tile t.  Here the only wait is the explicit one in front of the
// barrier that publishes the tile.
template <int IMM>
__device__ __forceinline__ void dma16(const unsigned char* base_uniform, unsigned voff,
                                      unsigned lds_addr_uniform) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, %2 offset:%3"
      :
      : "s"(lds_addr_uniform), "v"(voff), "s"(base_uniform), "n"(IMM)
      : "m0", "memory");
}

// The same with the lane's offset formed on the spot as (chunk ^ flip) + row: the K tile's
// chunk swizzle differs between a lane's four transfers by an XOR, and forming it here keeps
// the compiler from holding four precomputed offsets in registers through the main loop.
template <int IMM>
__device__ __forceinline__ void dma16_xor(const unsigned char* base_uniform, unsigned row_part,
                                          unsigned chunk_part, unsigned flip_uniform,
                                          unsigned lds_addr_uniform) {
  unsigned voff;
  asm volatile(
      "v_xad_u32 %0, %2, %3, %1\n\t"
      "s_mov_b32 m0, %4\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %5 offset:%6"
      : "=&v"(voff)
      : "v"(row_part), "v"(chunk_part), "s"(flip_uniform), "s"(lds_addr_uniform),
        "s"(base_uniform), "n"(IMM)
      : "m0", "memory");
}

// LOOP: when the append is done, with the tiles that fall to the workgroup as they pass through the loop, or with its
// share of the rows after it.  The loop wins where workgroups follow each other on a compute unit, and the rows at the
// end would keep the next one waiting: steps, end / loop, us: d 128, 256 units x 576 queries 107 / 101, 480 x 576
// 188 / 183, 256 x 300 37.9 / 36.7; d 64, 256 x 576 67.4 / 62.  Where all are resident at once it loses (80 x 576,
// d 128, 49.9 / 51.3; d 64, 32 x 1500 over 6000 kept rows 151 / 155), but not in the split form of head_dim 64 (64 x 400
// 27.6 / 26.7, 80 x 256 22.9 / 21.9; d 128 within 2 % either way), and it does in the wide form, whose barriers hold
// eight waves to the slowest store (4096 queries, 256 units, 2772 / 2796).  A form of its own: code that is not used
// costs 1-3 %.
template <int D, int WAVES, int SPLIT>
constexpr bool appends_in_loop(long long n_wg) {
  constexpr int kResident = 256 * Shape<D, WAVES, SPLIT>::kWavesPerSimd;  // plain form: workgroups on all compute units
  return WAVES == 4 && (SPLIT > 1 ? D == 64 : n_wg > kResident);
}

// What a launch writes besides its output: nothing, the second segment behind the first, or both segments, into a cache
// that is not the one it reads.
enum CopyWhat { kCopyNothing = 0, kCopySecond = 1, kCopyBoth = 2 };
struct CopyArgs {
  int what;  // CopyWhat
  uint16_t *k, *v;
  long long k_seq_stride, k_head_stride, v_seq_stride, v_head_stride;
};

template <int D, int WAVES, int SPLIT, bool LOOP>
__global__ __launch_bounds__(64 * WAVES * SPLIT)
__attribute__((amdgpu_waves_per_eu(Shape<D, WAVES, SPLIT>::kWavesPerSimd, Shape<D, WAVES, SPLIT>::kWavesPerSimd)))
void attend_pipe_kernel(const uint16_t* __restrict__ q, int n_q, const uint16_t* k, long long k_seq_stride,
                        long long k_head_stride, const uint16_t* v, long long v_seq_stride,
                        long long v_head_stride, int len1, const uint16_t* __restrict__ k2,
                        const uint16_t* __restrict__ v2, int len2, CopyArgs copy, int n_head,
                        int n_qtile, int n_wg, float scale_log2e, float no_max, uint16_t* __restrict__ out) {
  SCALEKV_STAMP(t_start);
#if defined(SCALEKV_TIMELINE)
  unsigned long long t_first_tile = 0;
  const unsigned long long c_start = __builtin_readcyclecounter();
#endif
  using G = Shape<D, WAVES, SPLIT>;
  constexpr int kStages = G::kStages, kRowBytes = G::kRowBytes, kTileBytes = G::kTileBytes;
  constexpr int NSL = G::kSlabs, NCB = G::kBlocks;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  const int wg = xcd_order(SCALEKV_WG_X, n_wg);  // all query tiles of a unit share one L2
  const int unit = wg / n_qtile, qtile = wg - unit * n_qtile;
  const int seq = unit / n_head, head = unit - seq * n_head;
  const int tid = threadIdx.x, lane = tid & 63;
  // wave `wave` of the `group`-th group: the groups share the query rows and take the key tiles in turn
  const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = SPLIT > 1 ? wave_id / WAVES : 0, wave = SPLIT > 1 ? wave_id - group * WAVES : wave_id;
  unsigned char* const k_lds = smem + group * (2 * kStages * kTileBytes);
  unsigned char* const v_lds = k_lds + kStages * kTileBytes;
  const int i = lane & 15, g = lane >> 4;
  const int q_base = qtile * G::kRows + wave * 32;
  const uint16_t* qu = q + (long long)unit * n_q * D;
  const unsigned char* ku = (const unsigned char*)(k + seq * k_seq_stride + head * k_head_stride);
  const unsigned char* vu = (const unsigned char*)(v + seq * v_seq_stride + head * v_head_stride);
  const unsigned char* k2u = (const unsigned char*)(k2 + (long long)unit * len2 * D);
  const unsigned char* v2u = (const unsigned char*)(v2 + (long long)unit * len2 * D);
  const int n_tile1 = (len1 + TN - 1) / TN;
  const int n_all = n_tile1 + (len2 + TN - 1) / TN;
  const int n_tile = (n_all - group + SPLIT - 1) / SPLIT;  // of this group
  const int n_turn = (n_all + SPLIT - 1) / SPLIT;          // of the first, which has the most

  // ---- tile loader: per thread kOps K vectors and kOps V vectors of 16 bytes (4 each; wide form and d 64: 2).
  // Instruction p of wave w fills LDS rows kWaveRows w + kRowsPerOp p .. (64 lanes x 16 B = 4 rows, d 64: 8);
  // the lane that lands in chunk slot s of row r fetches global chunk s ^ flip(r).  For this lane
  // r = r0 + kRowsPerOp p, and both flips are linear: its K chunk is c0 ^ k_step(p) with c0 the one for
  // p = 0 (bit 3 of r alone depends on p), and its V chunk does not depend on p.  One register pair serves all
  // instructions, the rest (1024 p bytes) rides in the instruction's immediate offset.
  const int ld_row = lane / G::kChunks;                                  // row inside an instruction
  const int ld_row0 = G::kWaveRows * wave + ld_row;
  const unsigned ld_krow = ld_row0 * kRowBytes;                          // K: row part
  const unsigned ld_kchunk = 16 * ((lane % G::kChunks) ^ G::k_flip(ld_row0));  // K: chunk part for p = 0
  const unsigned ld_vofs = ld_row0 * kRowBytes + 16 * ((lane % G::kChunks) ^ G::v_flip(ld_row0));
  constexpr auto k_step = [](int p) -> unsigned { return 16 * G::k_flip(G::kRowsPerOp * p); };  // bytes
  auto lds_addr = [](const unsigned char* p) -> unsigned {
    return (unsigned)(size_t)(const __attribute__((address_space(3))) unsigned char*)p;
  };
  // LDS byte addresses of this wave's 16 rows in stage 0 (wave-uniform, kept in scalar registers)
  const unsigned k_lds_wave = __builtin_amdgcn_readfirstlane(lds_addr(k_lds + G::kWaveRows * wave * kRowBytes));
  const unsigned v_lds_wave = __builtin_amdgcn_readfirstlane(lds_addr(v_lds + G::kWaveRows * wave * kRowBytes));
  // Tile t of the group: its number of valid rows, in whichever segment it lies.
  auto rows_of = [&](int t) {
    const int tile = t * SPLIT + group;
    return tile < n_tile1 ? len1 - tile * TN : len2 - (tile - n_tile1) * TN;
  };
  auto issue_k = [&](int t) __attribute__((always_inline)) {
    const unsigned dst = k_lds_wave + (t % kStages) * kTileBytes;
    const int tile = t * SPLIT + group;
    const unsigned char* src = tile < n_tile1 ? ku + (long long)tile * kTileBytes
                                              : k2u + (long long)(tile - n_tile1) * kTileBytes;
    const int valid = rows_of(t);
    if (valid >= TN) {
      // the immediate offset moves the LDS destination along with the global source, which
      // is exactly the kRowsPerOp rows between a lane's consecutive transfers
      dma16_xor<0>(src, ld_krow, ld_kchunk, 0u, dst);
      if constexpr (G::kOps >= 2) dma16_xor<1024>(src, ld_krow, ld_kchunk, k_step(1), dst);
      if constexpr (G::kOps == 4) {
        dma16_xor<2048>(src, ld_krow, ld_kchunk, k_step(2), dst);
        dma16_xor<3072>(src, ld_krow, ld_kchunk, k_step(3), dst);
      }
    } else {
      // ragged last tile: rows past the end re-read the last valid row (finite data that
      // the mask turns into zero weight).  (An opaque row number keeps what is formed from it in this branch.)
      int row0 = ld_row0;
      asm volatile("" : "+v"(row0));
#pragma unroll
      for (int p = 0; p < G::kOps; ++p) {
        const int back = max(row0 + G::kRowsPerOp * p - (valid - 1), 0) * kRowBytes;
        dma16<0>(src, row0 * kRowBytes + (ld_kchunk ^ k_step(p)) + 1024 * p - back, dst + 1024 * p);
      }
    }
  };
  auto issue_v = [&](int t) __attribute__((always_inline)) {
    const unsigned dst = v_lds_wave + (t % kStages) * kTileBytes;
    const int tile = t * SPLIT + group;
    const unsigned char* src = tile < n_tile1 ? vu + (long long)tile * kTileBytes
                                              : v2u + (long long)(tile - n_tile1) * kTileBytes;
    const int valid = rows_of(t);
    if (valid >= TN) {
      dma16<0>(src, ld_vofs, dst);
      if constexpr (G::kOps >= 2) dma16<1024>(src, ld_vofs, dst);
      if constexpr (G::kOps == 4) {
        dma16<2048>(src, ld_vofs, dst);
        dma16<3072>(src, ld_vofs, dst);
      }
    } else {
      int row0 = ld_row0;
      asm volatile("" : "+v"(row0));
#pragma unroll
      for (int p = 0; p < G::kOps; ++p) {
        const int back = max(row0 + G::kRowsPerOp * p - (valid - 1), 0) * kRowBytes;
        dma16<0>(src, ld_vofs + 1024 * p - back, dst + 1024 * p);
      }
    }
  };

  // ---- per-lane operand addresses (LDS, bytes) in the first 32-key block; key tile t is 4 rows further on
  unsigned k_adr[NSL];  // K operand, slab sl: chunk 4sl + g of the row that MFMA row i is fed
  {
    const int row = 16 * (i >> 2 & 1) + 8 * (i >> 3) + (i & 3);
#pragma unroll
    for (int sl = 0; sl < NSL; ++sl)
      k_adr[sl] = lds_addr(k_lds) + row * kRowBytes + 16 * ((4 * sl + g) ^ G::k_flip(row));
  }
  unsigned v_adr[NCB];  // V^T operand, channel block c: this lane's address role in the transposing load
  {
    const int row = 16 * (g & 1) + 8 * (g >> 1) + (i >> 2);
#pragma unroll
    for (int c = 0; c < NCB; ++c)
      v_adr[c] = lds_addr(v_lds) + row * kRowBytes + 16 * (2 * c ^ G::v_flip(row)) + 8 * (i & 3);
  }
  // (opaque, so that every load is one of these registers plus an immediate offset)
#pragma unroll
  for (int sl = 0; sl < NSL; ++sl) asm volatile("" : "+v"(k_adr[sl]));
#pragma unroll
  for (int c = 0; c < NCB; ++c) asm volatile("" : "+v"(v_adr[c]));

  // ---- Q fragments: B operand of the first product, resident for the whole kernel.  A lane's
  // fragments are 16-byte pieces of two query rows, 64 bytes apart: fetched as such, every
  // instruction of the wave would touch 16 rows with 64 bytes each.  Instead the wave's 32 rows
  // go, whole and 16 bytes per lane, straight into LDS and are read from there once the first
  // tile has arrived.  They wait in the last stages, which are not in use yet, each wave's rows exactly
  // where the same wave will later put its share of those tiles (kWaveRows K rows, then as many V rows,
  // kQParts such parts): nobody else writes there, so no barrier is needed before those
  // tiles are requested, only the wave's own reads must have returned.  Chunk c of row
  // r sits in slot c ^ q_flip(r), so that the fragment reads are free of bank conflicts.  Rows
  // past the end of the map repeat its last row; nothing is stored for them.
  bf16x8 qf[2][NSL];
  constexpr int kPartRows = G::kWaveRows, kQParts = 32 / kPartRows;
  auto q_part = [&](int part) -> unsigned char* {
    const int stage = kStages - kQParts / 2 + part / 2;
    return (part & 1 ? v_lds : k_lds) + stage * kTileBytes + kPartRows * wave * kRowBytes;
  };
  {
#pragma unroll
    for (int p = 0; p < G::kQOps; ++p) {
      const int r = G::kRowsPerOp * p + ld_row;
      const unsigned row = (unsigned)min(q_base + r, n_q - 1);
      const unsigned dst = __builtin_amdgcn_readfirstlane(lds_addr(q_part(p / G::kOps))) + 1024 * (p % G::kOps);
      dma16<0>((const unsigned char*)qu, row * kRowBytes + 16 * ((lane % G::kChunks) ^ G::q_flip(r)), dst);
    }
  }
  auto read_q = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int sl = 0; sl < NSL; ++sl)
        qf[b][sl] = *(const bf16x8*)((kPartRows == 16 ? q_part(b) : i < 8 ? q_part(2 * b) : q_part(2 * b + 1)) +
                                     (i % kPartRows) * kRowBytes + 16 * ((4 * sl + g) ^ G::q_flip(i)));
  };

  f32x4 o[2][NCB];   // [query tile][channel block]
  float neg_off[2];  // less the exponent offsets
  float l_run[2];    // this lane's share of the row sums

  typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  constexpr int kHalf = 32 * kRowBytes;
  constexpr int kSlots = 4 * NSL;          // MFMAs of one product over a block (the two have the same number)
  constexpr int kSteps = 16 / kSlots;      // softmax steps behind each
  static_assert(kSlots == 2 * NCB && 2 * NSL <= kSlots - kSlots / 2, "the requests fit in the slots");
  constexpr int kBarrierSlot = kSlots / 2 - 1;
  bf16x8 kf[2][NSL];       // K operand, [key tile][slab]
  s16x4 vf[NCB][2];        // V^T operand, [channel block][key tile]
  f32x4 sa[2][2], sb[2][2];  // scores of an even and an odd block, [query tile][key tile]
  u32x4 pa[2], pb[2];      // their weights, bf16

  auto read_k = [&](int ofs, int e) {
    kf[e & 1][e >> 1] = *(lds_bf16x8*)(k_adr[e >> 1] + ofs + 4 * (e & 1) * kRowBytes);
  };
  auto read_v = [&](int ofs, int e) {
    const unsigned adr = v_adr[e >> 1] + ofs + 4 * (e & 1) * kRowBytes;
    vf[e >> 1][e & 1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)adr);
  };
  // MFMA m of the two products over a block
  auto score_mfma = [&](f32x4 (&s)[2][2], int m) {
    const int sl = m >> 2, t = m >> 1 & 1, b = m & 1;
    const f32x4 sum = sl ? s[b][t] : f32x4{0.f, 0.f, 0.f, 0.f};
    s[b][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[t][sl], qf[b][sl], sum, 0, 0, 0);
  };
  auto value_mfma = [&](const u32x4 (&p)[2], int m) {
    const int c = m >> 1, b = m & 1;
    const bf16x8 vt = __builtin_bit_cast(bf16x8, __builtin_shufflevector(vf[c][0], vf[c][1], 0, 1, 2, 3, 4, 5, 6, 7));
    o[b][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt, __builtin_bit_cast(bf16x8, p[b]), o[b][c], 0, 0, 0);
  };
  // Step k of 32 of a block's softmax: four for each pair of weights.  (The empty statements keep each step in
  // its slot: without them the compiler moves the arithmetic to where its result is used.)
  auto softmax_step = [&](f32x4 (&s)[2][2], u32x4 (&p)[2], int k) {
    const int b = k >> 4, x = 2 * (k >> 2 & 3), t = x >> 2, v = x & 3;
    float w0 = s[b][t][v], w1 = s[b][t][v + 1];
#if defined(SCALEKV_ABLATE_SOFTMAX)
    if ((k & 3) == 3) p[b][x / 2] = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)w0, (__bf16)w1});
#else
    if ((k & 3) == 0) {
      w0 = fmaf(w0, scale_log2e, neg_off[b]);
      w1 = fmaf(w1, scale_log2e, neg_off[b]);
      asm volatile("" : "+v"(w0), "+v"(w1));
    } else if ((k & 3) == 1) {
      w0 = __builtin_amdgcn_exp2f(w0);
      asm volatile("" : "+v"(w0));
    } else if ((k & 3) == 2) {
      w1 = __builtin_amdgcn_exp2f(w1);
      asm volatile("" : "+v"(w1));
    } else {
      const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f}, pr = {(__bf16)w0, (__bf16)w1};
      uint32_t word = __builtin_bit_cast(uint32_t, pr);
      // the row sum adds the rounded weights, the very numbers the MFMA multiplies by
      l_run[b] = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, l_run[b], false);
      asm volatile("" : "+v"(word), "+v"(l_run[b]));
      p[b][x / 2] = word;
    }
    s[b][t][v] = w0;
    s[b][t][v + 1] = w1;
#endif
  };
  // hides the keys of a block (register v of key tile t = key 16(g & 1) + 8(g >> 1) + 4t + v) from `valid` on
  auto hide = [&](f32x4 (&s)[2][2], int valid) __attribute__((always_inline)) {
    if (valid < 32) {
      // (the lane group is taken from the lane number on the spot, so that the eight key
      // indices of this rarely taken branch are not kept in registers through the main loop)
      const int group = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)) >> 4;
      const int left = valid - 16 * (group & 1) - 8 * (group >> 1);
#pragma unroll
      for (int x = 0; x < 8; ++x)
        if (x >= left) s[0][x / 4][x % 4] = s[1][x / 4][x % 4] = -INFINITY;
    }
  };
  // largest score of each query of a block
  auto block_max = [&](const f32x4 (&s)[2][2], float (&mx)[2]) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      float m = s[b][0][0];
#pragma unroll
      for (int x = 1; x < 8; ++x) m = fmaxf(m, s[b][x / 4][x % 4]);
      mx[b] = xor32_max(xor16_max(m));
    }
  };

  // One product over a block, with the other work of the wave between its MFMAs: slot m is an MFMA, what
  // `beside` puts there, and kSteps steps of the softmax of another block.  The fences keep the order.
  auto slots = [&](auto mfma, auto beside, f32x4 (&s)[2][2], u32x4 (&p)[2],
                   int first_step) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < kSlots; ++m) {
      mfma(m);
      beside(m);
#pragma unroll
      for (int r = 0; r < kSteps; ++r) softmax_step(s, p, first_step + m * kSteps + r);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // ---- append in the loop: the second segment goes behind the first in the cache from the LDS, as its
  // tiles pass.  A wave copies the rows that it has brought in itself; turn x of the second segment falls to query tile
  // x mod n_qtile, so that the workgroups of a unit write at different times.
  // (Both segments: turn x falls to query tile x mod n_qtile from the first turn on.)
  [[maybe_unused]] unsigned char *kdu = nullptr, *vdu = nullptr;
  [[maybe_unused]] int copy_turn = -1;  // the next of this workgroup
  if constexpr (LOOP) {
    kdu = (unsigned char*)(copy.k + seq * copy.k_seq_stride + head * copy.k_head_stride);
    vdu = (unsigned char*)(copy.v + seq * copy.v_seq_stride + head * copy.v_head_stride);
    copy_turn = copy.what == kCopyBoth ? qtile : n_tile1 / SPLIT + qtile;
  }
  auto copy_tile = [&](int t, const unsigned char* stages, unsigned char* cache, auto ofs)
                       __attribute__((always_inline)) {
    const int tile = t * SPLIT + group;
    if (t >= n_tile || (tile < n_tile1 && copy.what != kCopyBoth)) return;
    // (formed on the spot, and a vector at a time: nothing of it stays in registers through the tile loop)
    const int mine = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const unsigned char* const src = stages + t % kStages * kTileBytes + G::kWaveRows * wave * kRowBytes + 16 * mine;
    const int row = tile < n_tile1 ? tile * TN : len1 + (tile - n_tile1) * TN;
    unsigned char* const dst = cache + (long long)row * kRowBytes;
    const int left = rows_of(t) - G::kWaveRows * wave - mine / G::kChunks;
#pragma unroll
    for (int p = 0; p < G::kOps; ++p) {
      const u32x4 val = *(const u32x4*)(src + 1024 * p);
      if (G::kRowsPerOp * p < left) __builtin_nontemporal_store(val, (u32x4*)(dst + ofs(p)));
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  [[maybe_unused]] auto copy_k = [&](int t) __attribute__((always_inline)) {
    copy_tile(t, k_lds, kdu, [&](int p) { return ld_krow + (ld_kchunk ^ k_step(p)) + 1024 * p; });
  };
  [[maybe_unused]] auto copy_v = [&](int t) __attribute__((always_inline)) {
    copy_tile(t, v_lds, vdu, [&](int p) { return ld_vofs + 1024 * p; });
  };
  // Publishes tile t + 1 of K and tile t of V, and requests the tiles kStages further on, in the place of those that
  // all waves have left.  Requests are made in the order V(x), K(x + 1): what may still be under way is those of x > t.
  auto turn = [&](int t) __attribute__((always_inline)) {
    if (kStages > 2 && t + kStages - 1 < n_tile)
      __builtin_amdgcn_s_waitcnt(0x0070 | 2 * (kStages - 2) * G::kOps);  // vmcnt; lgkmcnt(0)
    else
      __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
#if defined(SCALEKV_ABLATE_TRANSFER)
    if (t == 0 && kStages <= n_tile) issue_v(kStages - 1);  // (fills the last stage, where query rows have been)
#else
    if (t + kStages - 1 < n_tile) issue_v(t + kStages - 1);
    if (t + kStages < n_tile) issue_k(t + kStages);
#endif
    if constexpr (LOOP) {
      if (t == copy_turn) {
        copy_v(t);
        copy_turn += n_qtile;
      }
      if (t + 1 == copy_turn) copy_k(t + 1);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto nothing = [](int) {};
  // First half of tile t: softmax of its first block beside the scores of its second and the weighted values
  // of the block before.  st = t mod kStages.
  auto first_half = [&](int t, int st) __attribute__((always_inline)) {
    hide(sa, rows_of(t));
    __builtin_amdgcn_sched_barrier(0);
    slots([&](int m) { score_mfma(sb, m); },
          [&](int m) { read_v((st + kStages - 1) % kStages * kTileBytes + kHalf, m); },
          sa, pa, 0);
    slots([&](int m) { value_mfma(pb, m); },
          [&](int m) {
            if (m == kBarrierSlot) turn(t);
            const int e = m - kBarrierSlot - 1;
            if (e >= 0 && e < 2 * NSL) read_k((st + 1) % kStages * kTileBytes, e);
          },
          sa, pa, 16);
  };
  // Second half: softmax of its second block beside the scores of the next tile's first and the weighted values
  // of its own first.
  auto second_half = [&](int t, int st) __attribute__((always_inline)) {
    hide(sb, rows_of(t) - 32);
    __builtin_amdgcn_sched_barrier(0);
    slots([&](int m) { score_mfma(sa, m); }, [&](int m) { read_v(st * kTileBytes, m); },
          sb, pb, 0);
    slots([&](int m) { value_mfma(pa, m); },
          [&](int m) { if (m < 2 * NSL) read_k((st + 1) % kStages * kTileBytes + kHalf, m); },
          sb, pb, 16);
  };

  // ---- the pass without maxima
#pragma unroll
  for (int b = 0; b < 2; ++b) {
#pragma unroll
    for (int c = 0; c < NCB; ++c) o[b][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    l_run[b] = 0.f;
    neg_off[b] = -(no_max * scale_log2e);
  }
  if (SPLIT == 1 || n_tile > 0) {
    issue_k(0);
    issue_v(0);
  }
  if constexpr (kStages == 2) {
    if (SPLIT == 1 || n_tile > 0)
      __builtin_amdgcn_s_waitcnt(0x0f70 | G::kOps);  // vmcnt(kOps): all but the V tile
    else
      __builtin_amdgcn_s_waitcnt(0);
  } else if (n_tile > 1) {
    issue_k(1);
    issue_v(1);
    __builtin_amdgcn_s_waitcnt(0x0f70 | 3 * G::kOps);
  } else {
    __builtin_amdgcn_s_waitcnt(0);
  }
  __syncthreads();
#if defined(SCALEKV_TIMELINE)
  t_first_tile = __builtin_amdgcn_s_memrealtime();
#endif
  read_q();
#pragma unroll
  for (int e = 0; e < 2 * NSL; ++e) read_k(0, e);
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the query fragments are in registers, their space may be refilled
  if constexpr (kStages == 2) {
    if (n_tile > 1) issue_k(1);
  } else {
    if (n_tile > 2) issue_k(2), issue_v(2);
    if (n_tile > 3) issue_k(3);
  }
  if (LOOP && copy_turn == 0) copy_k(0);
  // (a wave whose query rows all lie behind the last one only carries its share of the tiles)
  const bool idle = q_base >= n_q || (SPLIT > 1 && n_tile == 0);
  int turns = 0;  // barriers of the tile loop behind this wave: all waves make n_turn
  if (!idle) {
#pragma unroll
    for (int m = 0; m < kSlots; ++m) score_mfma(sa, m);
#pragma unroll
    for (int e = 0; e < 2 * NSL; ++e) read_k(kHalf, e);
    hide(sa, rows_of(0));
#pragma unroll
    for (int m = 0; m < kSlots; ++m) score_mfma(sb, m);
    hide(sb, rows_of(0) - 32);
    {
      float mx[2], mx2[2];
      block_max(sa, mx);
      block_max(sb, mx2);
      bool grow = false;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        mx[b] = fmaxf(no_max, mx[b]);
        grow |= (mx2[b] - mx[b]) * scale_log2e > kRescaleThreshold;
      }
      const bool both = __builtin_amdgcn_ballot_w64(grow) != 0;
#pragma unroll
      for (int b = 0; b < 2; ++b) neg_off[b] = -((both ? fmaxf(mx[b], mx2[b]) : mx[b]) * scale_log2e);
    }
    __builtin_amdgcn_sched_barrier(0);
    slots(nothing, nothing, sa, pa, 0);
    turn(0);
    slots(nothing, [&](int m) { if (m < 2 * NSL) read_k(kTileBytes, m); }, sa, pa, 16);
    int t = 0;
    for (; t + kStages < n_tile; t += kStages) {
#pragma unroll
      for (int x = 0; x < kStages; ++x) {
        second_half(t + x, x);
        first_half(t + x + 1, (x + 1) % kStages);
      }
    }
#pragma unroll
    for (int x = 0; x < kStages - 1; ++x)
      if (t + 1 < n_tile) {
        second_half(t, x);
        first_half(t + 1, x + 1);
        ++t;
      }
    {
      const int ofs = t % kStages * kTileBytes;
      hide(sb, rows_of(t) - 32);
      slots(nothing, [&](int m) { read_v(ofs, m); }, sb, pb, 0);
      slots([&](int m) { value_mfma(pa, m); }, nothing, sb, pb, 16);
#pragma unroll
      for (int m = 0; m < kSlots; ++m) read_v(ofs + kHalf, m);
#pragma unroll
      for (int m = 0; m < kSlots; ++m) value_mfma(pb, m);
    }
    turns = n_tile;
  }
  if (SPLIT > 1 || idle)
    for (; turns < n_turn; ++turns) turn(turns);
  // A weight or a sum beyond the range, or inf or NaN in an accumulator (huge values times large weights)?  Weights are
  // not negative, so what went wrong with one is still in its row's sum; a sum of accumulators is finite only if they
  // all are (and may not be although they are: then the repeat is for nothing).
  bool overflowed = false;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    float largest = 0.f;
    f32x4 all = o[b][0];
#pragma unroll
    for (int c = 0; c < NCB; ++c) {
      if (c > 0) all += o[b][c];
#pragma unroll
      for (int v = 0; v < 4; ++v) largest = fmaxf(largest, fabsf(o[b][c][v]));
    }
    overflowed |= !(l_run[b] <= kRowSumLimit<SPLIT>) || !(fabsf(all[0] + all[1] + all[2] + all[3]) < INFINITY) ||
                  (SPLIT > 1 && largest > kSplitOutputLimit);
  }
  // ---- the pass that follows the maxima (every wave has left its last tile when the votes are in)
#if defined(SCALEKV_ABLATE_SOFTMAX)
  overflowed = false;
#endif
  if (__syncthreads_or(overflowed)) {
    float m_run[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
      for (int c = 0; c < NCB; ++c) o[b][c] = f32x4{0.f, 0.f, 0.f, 0.f};
      m_run[b] = no_max;
      l_run[b] = 0.f;
    }
    if (SPLIT == 1 || n_tile > 0) {
      issue_k(0);
      issue_v(0);
    }
    for (int t = 0; t < n_turn; ++t) {
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      if (t + 1 < n_tile) {
        issue_k(t + 1);
        issue_v(t + 1);
      }
      for (int half = idle || (SPLIT > 1 && t >= n_tile) ? 2 : 0; half < 2; ++half) {
        const int ofs = t % kStages * kTileBytes + half * kHalf;
#pragma unroll
        for (int e = 0; e < 2 * NSL; ++e) read_k(ofs, e);
#pragma unroll
        for (int e = 0; e < kSlots; ++e) read_v(ofs, e);
#pragma unroll
        for (int m = 0; m < kSlots; ++m) score_mfma(sa, m);
        hide(sa, rows_of(t) - 32 * half);
        float mx[2];
        block_max(sa, mx);
        bool grow = false;
#pragma unroll
        for (int b = 0; b < 2; ++b) grow |= (mx[b] - m_run[b]) * scale_log2e > kRescaleThreshold;
        if (__builtin_amdgcn_ballot_w64(grow) != 0) {
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const float m_new = fmaxf(m_run[b], mx[b]);
            const float alpha = __builtin_amdgcn_exp2f((m_run[b] - m_new) * scale_log2e);
            m_run[b] = m_new;
            l_run[b] *= alpha;
#pragma unroll
            for (int c = 0; c < NCB; ++c)
#pragma unroll
              for (int v = 0; v < 4; ++v) o[b][c][v] *= alpha;
          }
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) neg_off[b] = -(m_run[b] * scale_log2e);
#pragma unroll
        for (int k = 0; k < 32; ++k) softmax_step(sa, pa, k);
#pragma unroll
        for (int m = 0; m < kSlots; ++m) value_mfma(pa, m);
      }
    }
    __syncthreads();
  }
  SCALEKV_STAMP(t_loop_end);

  // ---- append at the end, first half: this workgroup's share of the second segment goes behind the first,
  // as 16-byte vectors.  The vectors of the first round (the whole share when it is at most 256
  // rows) are requested here, before the output is normalised and stored, so that their latency
  // hides behind that work; the registers of the operand fragments are free by now.
  const int ap_per = !LOOP && copy.what != kCopyNothing ? (len2 + n_qtile - 1) / n_qtile : 0;
  const int ap_row0 = min(qtile * ap_per, len2);
  const int ap_vec = min(ap_per, len2 - ap_row0) * (kRowBytes / 16);  // per tensor
  const u32x4* ap_ks = (const u32x4*)(k2u + (long long)ap_row0 * kRowBytes);
  const u32x4* ap_vs = (const u32x4*)(v2u + (long long)ap_row0 * kRowBytes);
  u32x4 ap_a[8], ap_b[8];
  // (a thread number of its own keeps the requests below the tile loop, and the row numbers of the store from
  // being held through it: they are those that the query rows were fetched with)
  int end_tid = tid;
  asm volatile("" : "+v"(end_tid));
  if (ap_vec > 0) {
    // (lanes past the end of the share re-read its last vector and store nothing)
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = min(u * G::kThreads + end_tid, ap_vec - 1);
      ap_a[u] = ap_ks[e];
      ap_b[u] = ap_vs[e];
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // ---- join the groups: a common offset, the largest, then the sums.  The group it comes from has a weight of about 1,
  // so that a part whose factor underflows (below 2^-126, of a sum below 2^102) is less than 2^-24 of the row.  Wave w of
  // the first group takes the parts that waves w of the others leave in LDS (the tile stages are free).
  constexpr int kPartBytes = 64 * 2 * NCB * 16;       // a wave's accumulators, fp32
  if constexpr (SPLIT > 1) {
    auto part = [&](int grp) { return (f32x4*)(smem + (grp - 1) * (WAVES * kPartBytes) + wave * kPartBytes) + lane; };
    __shared__ float part_off[SPLIT][WAVES][2][64], part_sum[SPLIT][WAVES][2][64];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      part_off[group][wave][b][lane] = -neg_off[b];
      part_sum[group][wave][b][lane] = l_run[b];
      if (group > 0)
#pragma unroll
        for (int c = 0; c < NCB; ++c) part(group)[(b * NCB + c) * 64] = o[b][c];
    }
    __syncthreads();
    if (group == 0) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        float top = -neg_off[b];
#pragma unroll
        for (int x = 1; x < SPLIT; ++x) top = fmaxf(top, part_off[x][wave][b][lane]);
        const float f0 = __builtin_amdgcn_exp2f(-neg_off[b] - top);
        l_run[b] *= f0;
#pragma unroll
        for (int c = 0; c < NCB; ++c) o[b][c] *= f0;
#pragma unroll
        for (int x = 1; x < SPLIT; ++x) {
          const float f = __builtin_amdgcn_exp2f(part_off[x][wave][b][lane] - top);
          l_run[b] += f * part_sum[x][wave][b][lane];
#pragma unroll
          for (int c = 0; c < NCB; ++c) o[b][c] += f * part(x)[(b * NCB + c) * 64];
        }
      }
    }
  }

  // ---- normalise and write.  A lane owns query columns i and 16 + i, channels 16c + 4g + v:
  // eight 8-byte pieces of each output row.  Stored from there, every instruction of the wave
  // would touch 16 rows with 32 bytes each; instead the wave turns its 32 x 128 block round in
  // LDS (the tile stages are free: every wave has left its last tile; each wave uses a region of
  // its own, rows padded to 272 bytes against bank conflicts) and writes whole 256-byte rows,
  // 16 bytes per lane, past the caches, which hold keys and values that other workgroups still want
  // (1024 queries x 1180 keys x 64 units after their pruning: 62.9 -> 61.0 us; with plain stores of the kept rows,
  // steps of 256 to 1024 queries are 2-8 % faster).  What reads the output next finds it in memory: a step and a
  // product of its whole output with a 128 x 512 matrix, us, past the caches / through them: 64 units x 256 queries
  // 45.5 / 45.3, 64 x 1024 95.8 / 96.2, 256 x 256 69.9 / 71.0, 256 x 576 185.4 / 182.2, 256 x 1024 339 / 342, 60 x 1215
  // 153.1 / 151.1, 256 x 4096 3109 / 3101: within 1.8 % either way; the step alone is 0-3 % faster past them.
  if (SPLIT == 1 || group == 0) {
    constexpr int kOutRowStride = kRowBytes + 16;
    const int end_lane = end_tid & 63;
    unsigned char* const ostage = smem + wave * (SPLIT > 1 ? kPartBytes : 32 * kOutRowStride);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const float inv = 1.f / xor32_sum(xor16_sum(l_run[b]));
#pragma unroll
      for (int c = 0; c < NCB; ++c) {
        const bf16x2 lo = {(__bf16)(o[b][c][0] * inv), (__bf16)(o[b][c][1] * inv)};
        const bf16x2 hi = {(__bf16)(o[b][c][2] * inv), (__bf16)(o[b][c][3] * inv)};
        uint2 pk;
        pk.x = __builtin_bit_cast(uint32_t, lo);
        pk.y = __builtin_bit_cast(uint32_t, hi);
        *(uint2*)(ostage + (16 * b + (end_lane & 15)) * kOutRowStride + 32 * c + 8 * (end_lane >> 4)) = pk;
      }
    }
    // the wave's own LDS writes have landed before it reads them back (same wave: no barrier)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int row0 = q_base;
    unsigned char* const obase = (unsigned char*)(out + ((long long)unit * n_q + row0) * D);
#pragma unroll
    for (int p = 0; p < G::kQOps; ++p) {
      const int r = G::kRowsPerOp * p + end_lane / G::kChunks, c = 16 * (end_lane % G::kChunks);
      const u32x4 val = *(const u32x4*)(ostage + r * kOutRowStride + c);
      if (row0 + r < n_q) __builtin_nontemporal_store(val, (u32x4*)(obase + (long long)r * kRowBytes + c));
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // ---- append, second half: store the first round, then whatever is left of a larger share.
  // The other workgroup on the compute unit keeps the matrix pipe busy meanwhile.
  if (ap_vec > 0) {
    // (copied here, the second segment goes behind the first where that is)
    u32x4* kd = (u32x4*)(const_cast<unsigned char*>(ku) + (long long)(len1 + ap_row0) * kRowBytes);
    u32x4* vd = (u32x4*)(const_cast<unsigned char*>(vu) + (long long)(len1 + ap_row0) * kRowBytes);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = u * G::kThreads + end_tid;
      if (e < ap_vec) {
        __builtin_nontemporal_store(ap_a[u], kd + e);
        __builtin_nontemporal_store(ap_b[u], vd + e);
      }
    }
    for (int e0 = 8 * G::kThreads; e0 < ap_vec; e0 += 8 * G::kThreads) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int e = e0 + u * G::kThreads + end_tid;
        if (e < ap_vec) { ap_a[u] = ap_ks[e]; ap_b[u] = ap_vs[e]; }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int e = e0 + u * G::kThreads + end_tid;
        if (e < ap_vec) {
          __builtin_nontemporal_store(ap_a[u], kd + e);
          __builtin_nontemporal_store(ap_b[u], vd + e);
        }
      }
    }
  }
#if defined(SCALEKV_TIMELINE)
  __builtin_amdgcn_s_waitcnt(0);  // the workgroup's stores have been issued and acknowledged
  if (tid == 0 && blockIdx.x < kTimelineMaxWg) {
    unsigned long long* rec = g_timeline + (long long)blockIdx.x * kTimelineWords;
    rec[0] = t_start;
    rec[1] = t_first_tile;
    rec[2] = t_loop_end;
    rec[3] = __builtin_amdgcn_s_memrealtime();
    rec[4] = __builtin_amdgcn_s_getreg((31 << 11) | 4);  // HW_ID: compute unit, shader array, shader engine
    rec[5] = c_start;
    rec[6] = __builtin_readcyclecounter();
  }
#endif
}

template <int D, int WAVES, int SPLIT, bool LOOP>
hipError_t launch_form(int n_unit, int n_head, const void* q, int n_q, KvView k, KvView v, int len1, const void* k2,
                       const void* v2, int len2, const CopyArgs& copy, float sm_scale, void* out, hipStream_t stream,
                       hipEvent_t start, hipEvent_t stop) {
  using G = Shape<D, WAVES, SPLIT>;
  constexpr int kLds = kLdsBytes<D, WAVES, SPLIT>;
  const auto kernel = attend_pipe_kernel<D, WAVES, SPLIT, LOOP>;
  static std::atomic<uint64_t> configured{0};
  const hipError_t e = allow_dynamic_lds((const void*)kernel, kLds, configured);
  if (e != hipSuccess) return e;
  const float scale_log2e = sm_scale * 1.4426950408889634f;
  const float no_max = no_maximum(scale_log2e);
  const int n_qtile = (n_q + G::kRows - 1) / G::kRows;
  const int n_wg = n_qtile * n_unit;
  if (start || stop)
    hipExtLaunchKernelGGL(kernel, dim3(n_wg), dim3(G::kThreads), kLds, stream, start, stop, 0, (const uint16_t*)q, n_q,
                          (const uint16_t*)k.ptr, k.seq_stride, k.head_stride, (const uint16_t*)v.ptr, v.seq_stride,
                          v.head_stride, len1, (const uint16_t*)k2, (const uint16_t*)v2, len2, copy, n_head, n_qtile, n_wg,
                          scale_log2e, no_max, (uint16_t*)out);
  else
    hipLaunchKernelGGL(kernel, dim3(n_wg), dim3(G::kThreads), kLds, stream, (const uint16_t*)q, n_q,
                       (const uint16_t*)k.ptr, k.seq_stride, k.head_stride, (const uint16_t*)v.ptr, v.seq_stride,
                       v.head_stride, len1, (const uint16_t*)k2, (const uint16_t*)v2, len2, copy, n_head, n_qtile, n_wg,
                       scale_log2e, no_max, (uint16_t*)out);
  return hipGetLastError();
}

template <int D, int WAVES, int SPLIT>
hipError_t launch(int n_unit, int n_head, const void* q, int n_q, KvView k, KvView v, int len1, const void* k2,
                  const void* v2, int len2, const CopyArgs& copy, float sm_scale, void* out, hipStream_t stream,
                  hipEvent_t start, hipEvent_t stop) {
  constexpr int kRows = Shape<D, WAVES, SPLIT>::kRows;
  const bool loop = copy.what == kCopyBoth ||
                    (copy.what == kCopySecond &&
                     appends_in_loop<D, WAVES, SPLIT>((long long)n_unit * ((n_q + kRows - 1) / kRows)));
  return loop ? launch_form<D, WAVES, SPLIT, true>(n_unit, n_head, q, n_q, k, v, len1, k2, v2, len2, copy, sm_scale, out,
                                                   stream, start, stop)
              : launch_form<D, WAVES, SPLIT, false>(n_unit, n_head, q, n_q, k, v, len1, k2, v2, len2, copy, sm_scale, out,
                                                    stream, start, stop);
}

}  // namespace

hipError_t launch_attend_pipe(int n_unit, int n_head, int d, const void* q, int n_q, KvView k, KvView v,
                              int len1, const void* k2, const void* v2, int len2, const AttendCopy* copy_to,
                              float sm_scale, void* out, hipStream_t stream, hipEvent_t start,
                              hipEvent_t stop) {
  CopyArgs copy{};
  if (copy_to) {
    copy.what = copy_to->both ? kCopyBoth : kCopySecond;
    copy.k = (uint16_t*)const_cast<void*>(copy_to->k.ptr); copy.v = (uint16_t*)const_cast<void*>(copy_to->v.ptr);
    copy.k_seq_stride = copy_to->k.seq_stride; copy.k_head_stride = copy_to->k.head_stride;
    copy.v_seq_stride = copy_to->v.seq_stride; copy.v_head_stride = copy_to->v.head_stride;
  }
#define SCALEKV_PIPE(D, W, S) \
  launch<D, W, S>(n_unit, n_head, q, n_q, k, v, len1, k2, v2, len2, copy, sm_scale, out, stream, start, stop)
  switch (pipe_form(d, n_unit, n_q, len1 + len2)) {
    case PipeForm::kWide: return SCALEKV_PIPE(128, 8, 1);
    case PipeForm::kSplit: return d == 128 ? SCALEKV_PIPE(128, 4, 2) : SCALEKV_PIPE(64, 4, 3);
    default: return d == 128 ? SCALEKV_PIPE(128, 4, 1) : SCALEKV_PIPE(64, 4, 1);
  }
#undef SCALEKV_PIPE
}

}  // namespace scalekv

#if defined(SCALEKV_TIMELINE)
// Measurement-only builds: copies the records of workgroups 0 .. n_wg-1 of the most recent
// attend_pipe_kernel launch (kTimelineWords words each) to host memory.  Synchronises the device.
extern "C" int scalekv_timeline_read(unsigned long long* dst, int n_wg) {
  if (!dst || n_wg < 0 || n_wg > scalekv::kTimelineMaxWg) return -1;
  if (hipDeviceSynchronize() != hipSuccess) return -2;
  return hipMemcpyFromSymbol(dst, HIP_SYMBOL(scalekv::g_timeline),
                             sizeof(unsigned long long) * scalekv::kTimelineWords * n_wg) == hipSuccess ? 0 : -2;
}
#endif
