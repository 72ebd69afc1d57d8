// Heads whose vocabulary does not fill the chip: the product is cut along the hidden dimension too.
//
// A row block of 128 weight rows is one workgroup of the heads' kernels, so a head of a few thousand rows leaves most of the
// 256 compute units idle while each workgroup walks the whole hidden dimension (4096 elements: 32 steps of 0.4 to 1 us).
// Here a workgroup takes one of `splits` ranges of the hidden dimension of a 128-row block and of up to 16, 32, 64 or 128
// columns, and leaves its sums as part[split][column][row]; the kernel that follows holds a whole column in one workgroup,
// adds the ranges in ascending order and finishes it (top-k and log-sum-exp, or the best token): two launches, as before.
// Equal weight rows still give equal logits - every row is cut at the same places.
//
// Which way: plan_head compares what both are made of.  A step of a tile takes what its LDS traffic takes (0.35 us for 16
// columns to 1.1 for 128; float: the matrix rate, 0.45 to 3.5), or its share of the weights' stream.  Measured, a whole
// call in a HIP graph before / with ranges, us:
//   base head, bf16:  128 columns x 1565 rows of 3328  37.0 / 14.9     128 x 6189 of 4096 (2 sequences)  65.4 / 34.0
//     64 x 3249 of 4072  34.1 / 24.0     512 x 1030 of 768 float  101.2 / 19.2     128 x 10407 of 2816  35.0 / 35.0 (not taken;
//     with three ranges 37.4: 16 MB of partial sums)
//   draft head, bf16:  40 columns x 2235 of 4096, k = 8  44.4 / 18.9     7 x 3801 of 4456  34.7 / 25.1     float:  30 x 2215 of
//     512  33.9 / 14.6     a step of 128 rows and 8 slots, 3176 x 4833  152 / 91
// 60 drawn calls each: draft head 1.29, base head 1.60 times as fast in the mean, the slowest 0.98 (within the scatter).
#pragma once

#include "common.h"

namespace ctcspec {

constexpr int kHeadMaxSplits = 16;
constexpr int kHeadColumnThreads = 512;                      // of the kernels that finish a column
constexpr int kHeadMaxRows = kHeadColumnThreads * 4 * 8;     // vocabulary rows they hold
// room for partial sums: the draft head's (the context's and the static scratch of the entry point that allocates nothing
// alike, so that both take the same way) and the base head's
constexpr size_t kDraftPartFloats = (size_t)2 << 20, kHeadPartFloats = (size_t)4 << 20;

struct HeadRangeParams {
  const void* hidden;  // [cols][D]
  const void* w;       // [V][D]
  const void* zeros;   // 256 bytes of zeros
  float* part;         // [splits][cols][row_blocks * 128]
  int cols, D, V;
  int tile_cols;       // 16, 32, 64 or 128
  int splits;
  int row_blocks, col_blocks;
};

// whole_us: what the way without ranges takes, by head_whole_us.  Fills tile_cols and splits; false: not worth it.
bool plan_head(HeadRangeParams& p, bool f32, double whole_us, double finish_us, size_t part_floats);
// the heads' own kernels: `rows` x `tile_cols` tiles over all steps, `finish_us` of epilogue
double head_whole_us(int V, int cols, int D, bool f32, int rows, int tile_cols, double finish_us);
hipError_t launch_head_ranges(const HeadRangeParams& p, bool f32, hipStream_t stream);
hipError_t prepare_head_ranges();

#if defined(__HIPCC__)
// A column's logits by a workgroup of kHeadColumnThreads: the ranges' sums in ascending order; z[j] holds rows
// 4 (j * threads + tid) .. + 3, what lies behind the row blocks is left at 0.
template <int NV>
__device__ __forceinline__ void load_head_column(const HeadRangeParams& p, int col, f32x4 (&z)[NV]) {
  const int Vp = p.row_blocks * kRowsPerBlock, tid = threadIdx.x;
  const float* src = p.part + (size_t)col * Vp;
  const size_t stride = (size_t)p.cols * Vp;
#pragma unroll
  for (int j = 0; j < NV; ++j) z[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
  for (int s = 0; s < p.splits; ++s) {
    f32x4 x[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int r = 4 * (j * kHeadColumnThreads + tid);
      x[j] = *(const f32x4*)(src + s * stride + (r < Vp ? r : 0));
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) z[j] += x[j];
  }
}
// the column's logits to a row of the output, which starts at any element
template <int NV>
__device__ __forceinline__ void store_head_column(float* out, int V, const f32x4 (&z)[NV]) {
  struct PackedF4 { f32x4 v; } __attribute__((packed, aligned(4)));
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int r = 4 * (j * kHeadColumnThreads + (int)threadIdx.x);
    if (r + 3 < V) {
      ((PackedF4*)(out + r))->v = z[j];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (r + i < V) out[r + i] = z[j][i];
    }
  }
}
// instantiates a column kernel for the rows it has to hold
template <typename F>
static hipError_t launch_for_rows(int V, F&& launch) {
  if (V <= 4 * kHeadColumnThreads) return launch(std::integral_constant<int, 1>{});
  if (V <= 8 * kHeadColumnThreads) return launch(std::integral_constant<int, 2>{});
  if (V <= 16 * kHeadColumnThreads) return launch(std::integral_constant<int, 4>{});
  return launch(std::integral_constant<int, 8>{});
}
#endif

}  // namespace ctcspec
