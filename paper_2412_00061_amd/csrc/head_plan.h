// Which way a head takes (ctc_draft_topk, verify_head_argmax): its own kernel, or the product cut along the hidden dimension
// (head_ranges.h).  Host code without HIP, so that a test can ask it.
//
// plan_head compares what both are made of; both take a second launch.  A step of a tile takes what its LDS traffic takes
// (0.35 us for 16 columns to 1.1 for 128; float: the matrix rate, 0.45 to 3.5), or its share of the weights' stream.  The
// kernel that finishes a column gets slower where a thread holds eight groups of rows: a draft head of 8193 to 16384 rows
// takes 4 to 5 us longer so than with its own epilogue and merge, at the same product (up to 8192 rows 1.4, up to 4096 0.9 less), a
// base head 4 (2.3, 1.7).  Measured, a whole call in a HIP graph before / with ranges, us:
//   base head, bf16:  128 columns x 1565 rows of 3328  37.0 / 14.9     128 x 6189 of 4096 (2 sequences)  65.4 / 34.0
//     64 x 3249 of 4072  34.1 / 24.0     512 x 1030 of 768 float  101.2 / 19.2     128 x 10407 of 2816  35.0 / 35.0 (not taken;
//     with three ranges 37.4: 16 MB of partial sums)     85 x 9043 of 2040  32.7 / 35.5 (not taken)
//   draft head, bf16:  40 columns x 2235 of 4096, k = 8  44.4 / 18.9     7 x 3801 of 4456  34.7 / 25.1     float:  30 x 2215 of
//     512  33.9 / 14.6     18 x 10174 of 768  24.8 / 28.3 (not taken)     a step of 128 rows and 8 slots, 3176 x 4833  152 / 91
//   draft head, bf16, 8 columns of 4096 (the streaming kernel's):  501 rows 23.9 / 13.3     2001  20.5 / 13.1     4001  23.7 / 18.6
//     6001  25.5 / 24.1 with two (not taken; the model sees 2 %).  With the merge left to ctc_collapse_tree, both calls together,
//     4001 rows: 44.7 with a merge of its own, 47.4 with a deferred one, 39.1 with ranges - no reason for another line there,
//     and a call takes the same way, to the same bits, whether the merge is deferred or not.
// The steps' times are those of the loop through registers (gemm_tile.h).  4098 calls drawn, every plan timed with the loops that run now:
// with this rule 0.72 of the time without ranges in the mean, 18 more than 2 % slower than without (the worst 288 columns x 10360 rows of
// 3328, 61.7 us against 45.4), 8.5 % above the best plan of each.
#pragma once

#include <stddef.h>

namespace ctcspec {

constexpr int kHeadRowBlock = 128;                           // vocabulary rows of a workgroup
constexpr int kHeadColBlock = 128;                           // columns of the base head's own kernel
constexpr int kHeadMaxSplits = 16;
constexpr int kHeadColumnThreads = 512;                      // of the kernels that finish a column
constexpr int kHeadMaxRows = kHeadColumnThreads * 4 * 8;     // vocabulary rows they hold
// partial sums that a call may leave: the draft head's (in a context and in the static scratch of the entry point that allocates
// nothing alike, so that both take the same way) and the base head's
constexpr size_t kDraftPartFloats = (size_t)2 << 20, kHeadPartFloats = (size_t)4 << 20;
// room for the sums of every call with up to `cols` columns and `vocab_rows` rows (a context's limits); `most` is one of those above
inline size_t head_part_floats(long long cols, int vocab_rows, size_t most) {
  const int rows = vocab_rows < kHeadMaxRows ? vocab_rows : kHeadMaxRows;
  const size_t all = (size_t)kHeadMaxSplits * cols * ((rows + kHeadRowBlock - 1) / kHeadRowBlock * kHeadRowBlock);
  return all < most ? all : most;
}

// Whether `bytes` of weights are read by nontemporal loads (dma_tile.h): rows of whole cache lines, unless a program that small may
// find them in the 256 MB last-level cache.  32000 rows, us plain / nontemporal, first when the same weights come again and
// again, then when others went through in between:
//   16 columns:  33 MB 9.5 / 11.5, 12.6 / 11.8     49 MB 12.6 / 13.2, 14.7 / 13.8     66 MB 15.6 / 15.4, 16.9 / 16.1
//     131 MB 23.6 / 25.3, 29.6 / 26.6     262 MB 42.3 / 44.5, 51.8 / 45.5     328 MB 57.2 / 52.1, 58.8 / 52.6
//   8 columns of 4096, 8001 rows (66 MB): 23.9 / 28.8, 30.1 / 28.3     128 columns, 262 MB: 51.5 / 52.0, 58.0 / 52.2
// Other rows share lines with their neighbours and with the next step, and nontemporal loads fetch those again: rows of 4104
// elements, 16 columns 41.7 / 53.9, 50.2 / 55.0; 128 columns 56.8 / 65.6, 64.2 / 66.2.
// 48 MB is a middle: where all else goes through in between, nontemporal loads are up to 7 % faster below it as well; 600 calls drawn, three
// states in turn, are 0.9 to 3.6 % slower with them in the mean, up to 27 %.
inline bool streamed_weights(long long bytes, long long row_bytes) { return row_bytes % 128 == 0 && bytes > (48LL << 20); }

// Which loop a head's tiles take, in `splits` ranges of its hidden dimension: the one that loads straight into LDS (dma_tile.h), or the one
// through registers (gemm_tile.h).  The former takes rows that start at multiples of 16 bytes (the row size is one), 256 of them within
// 32-bit offsets.  With a single step of 256 bytes, whole rows or ranges, or a single row block there is nothing to pipeline, and the way
// through registers is 0.3 to 0.5 us shorter: 100 rows of 64 float, 64 and 128 columns 6.3 us so, 6.7 straight into LDS alone; rows of 256
// bf16, 2000 of them, 7 to 10 % faster so; 975 rows of 256 float in four ranges, 20 columns 6.7 and 7.1, 465 rows, 32 columns 10.9 and 11.4.
inline bool rows16(int D, int elem) { return ((long long)D * elem) % 16 == 0 && (long long)D * elem * 256 < (1LL << 32); }
inline bool dma_rows(long long V, int D, int elem, int splits = 1) {
  return rows16(D, elem) && (long long)D * elem > 256LL * splits && V > kHeadRowBlock;
}

struct HeadPlan {
  int cols, D, V;
  int tile_cols;       // 16, 32, 64 or 128
  int splits;
  int row_blocks, col_blocks;
};

constexpr double kHeadMergeUs = 2.0;  // the second launch, which a single row block does not take
constexpr double kStartUs = 6.0;  // a workgroup's way to its first step
inline double step_us(int tile_cols, bool f32, long long groups) {
  const int i = tile_cols <= 16 ? 0 : tile_cols <= 32 ? 1 : tile_cols <= 64 ? 2 : 3;
  static const double lds[4] = {0.35, 0.4, 0.9, 1.1}, mfma[4] = {0.45, 0.9, 1.75, 3.5};
  const double own = f32 ? mfma[i] : lds[i], stream = (double)(groups < 256 ? groups : 256) * 32768.0 / 5.9e6;
  return own > stream ? own : stream;
}
inline double walk_us(long long groups, double steps, double step) {
  return (double)((groups + 255) / 256) * (kStartUs + steps * step);
}
// the heads' own kernels: `rows` x `tile_cols` tiles over all steps, `finish_us` of epilogue
inline double head_whole_us(int V, int cols, int D, bool f32, int rows, int tile_cols, double finish_us) {
  const long long groups = (long long)((V + rows - 1) / rows) * ((cols + tile_cols - 1) / tile_cols);
  const double steps = (double)D * (f32 ? 4 : 2) / 256.0;
  return walk_us(groups, steps, step_us(tile_cols, f32, groups) * rows / 128.0) + finish_us;
}
// whole_us: what the way without ranges takes, by head_whole_us.  Fills tile_cols and splits; false: not worth it.
inline bool plan_head(HeadPlan& p, bool f32, double whole_us, double finish_us, size_t part_floats) {
  if (p.V > kHeadMaxRows) return false;
  p.row_blocks = (p.V + kHeadRowBlock - 1) / kHeadRowBlock;
  const double steps = (double)p.D * (f32 ? 4 : 2) / 256.0;
  const size_t sums = (size_t)p.cols * p.row_blocks * kHeadRowBlock;  // of one range
  double least = 0.9 * whole_us - 0.43;  // (the model is not better than that)
  p.splits = 0;
  for (int tile = 16; tile <= 128; tile *= 2) {
    const long long groups = (long long)p.row_blocks * ((p.cols + tile - 1) / tile);
    for (int S = 1; S <= kHeadMaxSplits && (S == 1 || S <= steps) && S * sums <= part_floats; ++S) {
      const double us = walk_us(groups * S, steps / S, step_us(tile, f32, groups * S)) + (double)S * sums * 8.0 / 3e6 +
                        finish_us + ((p.cols + 255) / 256) * (double)S * p.V * 4.0 / 45e3;
      if (us < least) {
        least = us;
        p.splits = S;
        p.tile_cols = tile;
      }
    }
    if (tile >= p.cols) break;
  }
  if (p.splits == 0) return false;
  p.col_blocks = (p.cols + p.tile_cols - 1) / p.tile_cols;
  return true;
}

// Base head, more than 128 columns, rows on 16-byte boundaries: 256-row tiles of 256 columns (a step 1.7 times that of 128 columns:
// 103 us against 60 for a round over the compute units at 4096) or of 128, by the rounds that they take.  215 shapes (512 to 5120 elements a
// row, float to 1024, 2000 to 50000 rows, 160 to 512 columns), both timed: within 3 % of the better one but for 300 and 384 columns x 50000 rows of
// 3000 (187 / 162 us, 202 / 169).
inline int head_wide_columns(int V, int cols) {
  const long long rows = (V + 255) / 256;
  const long long rounds256 = (rows * ((cols + 255) / 256) + 255) / 256, rounds128 = (rows * ((cols + 127) / 128) + 255) / 256;
  return 17 * rounds256 <= 10 * rounds128 ? 256 : 128;
}
inline int head_tile_cols(int cols) { return cols <= 16 ? 16 : cols <= 32 ? 32 : cols <= 64 ? 64 : 128; }
// what the epilogues take: joining the wavefronts' k-lists; a column's workgroup pops k keys, and is slow with eight groups of
// rows a thread
constexpr int kHeadSlowRows = kHeadColumnThreads * 4 * 4;
inline bool plan_draft_head(HeadPlan& p, bool f32, int k) {
  const int tile_cols = head_tile_cols(p.cols);
  const double epilogue_us = tile_cols == 16 ? 1.5 : k <= 2 ? 2.0 : k <= 4 ? 3.0 : 4.0;
  // (the epilogue of a lane per column takes as long as the launch that it saves)
  const double merge_us = p.V <= kHeadRowBlock && tile_cols == 16 ? -0.5 * kHeadMergeUs : 0.0;
  return plan_head(p, f32, head_whole_us(p.V, p.cols, p.D, f32, kHeadRowBlock, tile_cols, epilogue_us) + merge_us,
                   1.5 + 0.2 * k + (p.V > kHeadSlowRows ? 3.0 : 0.0), kDraftPartFloats);
}
inline bool plan_base_head(HeadPlan& p, bool f32) {
  const int rows = p.cols > kHeadColBlock ? 256 : 128;
  // a single row block, one workgroup for 16 columns, is slower a step than many: float, 6 steps 8.2 us, 8.5 9.7, 16 14.0, 32 23.9 (in eight ranges
  // 8.2, 8.7, 10.5, 10.9; by the others' step it was not cut at 8.5)
  const double alone_us = f32 ? 5.3 + 0.61 * ((double)p.D * 4 / 256.0) : head_whole_us(p.V, p.cols, p.D, f32, kHeadRowBlock, 16, 1.0) - kHeadMergeUs;
  const double whole_us = p.V <= kHeadRowBlock ? alone_us : head_whole_us(p.V, p.cols, p.D, f32, rows, head_tile_cols(p.cols), 1.0);
  return plan_head(p, f32, whole_us,
                   p.V > kHeadSlowRows ? 3.0 : 1.0, kHeadPartFloats);
}

// ---- the draft head's streaming kernel (bf16) -----------------------------------------------------------------------
// bytes per staged W row: 256 bf16 + pad.  The LDS serves a 16-byte access 16 lanes at a time - lanes l .. l+7 with
// l+16 .. l+23 - so a fragment read (lane = row c, chunk g) is conflict-free when rows c .. c+7 at chunks g and g+1
// fall on 16 different groups of 4 banks: pitch = 32 mod 64 bytes (with 16 bytes of pad the conflict counter read
// 8200 cycles per workgroup)
constexpr int kWRowStride = 512 + 32;
constexpr int kWStageBytes = 16 * kWRowStride;  // per wave
constexpr int kMfmaWaves = 8;
constexpr int kMfmaLdsLimit = 160 * 1024 - 64;                          // dynamic LDS that the kernel may ask for
// Register stages of its prefetch, 0: not taken.  It needs the hidden states of all columns in LDS over the whole hidden
// dimension (4 stages; 2 when D is a multiple of 512 but not of 1024).  A stream of one workgroup is none: 64 columns x 100 rows of 512
// 15.9 us, 12.8 as a tile, 7.7 in the ranges it gets.
inline int draft_stream_stages(int cols, int D, int vocab_rows) {
  if (vocab_rows <= kHeadRowBlock || (long long)cols * (2LL * D + 32) > kMfmaLdsLimit - kMfmaWaves * kWStageBytes) return 0;
  return D % 1024 == 0 ? 4 : D % 512 == 0 ? 2 : 0;
}

}  // namespace ctcspec
