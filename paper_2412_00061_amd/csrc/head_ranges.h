// Heads whose vocabulary does not fill the chip: the product is cut along the hidden dimension too.
//
// A row block of 128 weight rows is one workgroup of the heads' kernels, so a head of a few thousand rows leaves most of the
// 256 compute units idle while each workgroup walks the whole hidden dimension (4096 elements: 32 steps of 0.4 to 1 us).
// Here a workgroup takes one of `splits` ranges of the hidden dimension of a 128-row block and of up to 16, 32, 64 or 128
// columns, and leaves its sums as part[split][column][row]; the kernel that follows holds a whole column in one workgroup,
// adds the ranges in ascending order and finishes it (top-k and log-sum-exp, or the best token): two launches, as before.
// Equal weight rows still give equal logits - every row is cut at the same places.
#pragma once

#include "common.h"
#include "head_plan.h"

namespace ctcspec {

static_assert(kHeadRowBlock == kRowsPerBlock && kHeadColBlock == kVerifyCols, "the rule's blocks are the kernels'");

struct HeadRangeParams : HeadPlan {
  const void* hidden;  // [cols][D]
  const void* w;       // [V][D]
  const void* zeros;   // 256 bytes of zeros
  float* part;         // [splits][cols][row_blocks * 128]
  bool streamed;       // streamed_weights
};

hipError_t launch_head_ranges(const HeadRangeParams& p, bool f32, hipStream_t stream);
hipError_t prepare_head_ranges();

#if defined(__HIPCC__)
// A column's logits by a workgroup of kHeadColumnThreads: the ranges' sums in ascending order; z[j] holds rows
// 4 (j * threads + tid) .. + 3.  What lies behind the row blocks holds another row's sums: the caller leaves rows >= V out.
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
