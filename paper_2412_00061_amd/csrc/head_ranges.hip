// The product of a head cut into ranges of the hidden dimension (head_ranges.h; head_plan.h has the rule that chooses it).
#include <type_traits>

#include "dma_tile.h"
#include "head_ranges.h"

namespace ctcspec {

// Bound: start-up (a workgroup's first tile is in LDS after about 6 us) and then a step's way from HBM or L2 into LDS (dma_tile.h); the
// partial sums go out in 64-byte pieces, nontemporal (read once, by another kernel).
template <typename SH, typename EL>
__global__ __launch_bounds__(64 * kTileWaves) void head_range_kernel(HeadRangeParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  static_assert(SH::ROWS == kRowsPerBlock, "row blocks of 128");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave / SH::WC, wc = wave % SH::WC;
  const int c = lane & 15, g = lane >> 4;
  // the column blocks of a (row block, range) run on one XCD, side by side (verify_head.hip has the reason)
  const int slot = blockIdx.x >> 3, unit = (slot / p.col_blocks) * 8 + (blockIdx.x & 7);
  if (unit >= p.row_blocks * p.splits) return;
  const int cb = slot % p.col_blocks, rb = unit % p.row_blocks, split = unit / p.row_blocks;
  const int col0 = cb * SH::COLS, cols = p.cols - col0 < SH::COLS ? p.cols - col0 : SH::COLS;
  // ranges of whole steps - of whole trips of the tile loop where there are enough - and the last one takes the rest
  const size_t row_bytes = (size_t)p.D * EL::ELEM;
  const int steps = (int)(row_bytes / SH::STEPB);
  const int per = steps >= 4 * p.splits ? 4 : 1;
  const int t0 = split * (steps / per) / p.splits * per, t1 = (split + 1) * (steps / per) / p.splits * per;
  const size_t from = (size_t)t0 * SH::STEPB, to = split + 1 == p.splits ? row_bytes : (size_t)t1 * SH::STEPB;
  GemmTileArgs t;
  t.w = (const unsigned char*)p.w + from;
  t.hidden = (const unsigned char*)p.hidden + (size_t)col0 * row_bytes + from;
  t.zeros = p.zeros; t.D = (int)((to - from) / EL::ELEM); t.pitch = p.D; t.V = p.V; t.row_base = rb * SH::ROWS; t.streamed = p.streamed;
  f32x4 acc[SH::RT][SH::CTW];
  tile_product<SH, EL>(t, TileColumns{cols}, smem, acc);
  const int Vp = p.row_blocks * SH::ROWS;
  float* out = p.part + ((size_t)split * p.cols + col0) * Vp + t.row_base;
#pragma unroll
  for (int ct = 0; ct < SH::CTW; ++ct) {
    const int col = (wc * SH::CTW + ct) * 16 + c;
    if (col >= cols) continue;
#pragma unroll
    for (int rt = 0; rt < SH::RT; ++rt)
      __builtin_nontemporal_store(acc[rt][ct], (f32x4*)(out + (size_t)col * Vp + (wr * SH::RT + rt) * 16 + g * 4));
  }
}

template <typename F>
static hipError_t each_shape(bool dma, bool aligned, F&& f) {
  auto one = [&](auto straight, auto tile) { return dma ? f(straight) : aligned ? f(Rows16<decltype(tile)>{}) : f(tile); };
  hipError_t e = one(Dma128x16{}, Tile128x16{});
  if (e == hipSuccess) e = one(Dma128x32{}, Tile128x32{});
  if (e == hipSuccess) e = one(Dma128x64{}, Tile128x64{});
  if (e == hipSuccess) e = one(Dma128x128{}, Tile128x128{});
  return e;
}
template <typename EL>
static hipError_t launch_type(const HeadRangeParams& p, hipStream_t stream) {
  return each_shape(dma_rows(p.V, p.D, EL::ELEM, p.splits), rows16(p.D, EL::ELEM), [&](auto shape) {
    using SH = decltype(shape);
    if (SH::COLS != p.tile_cols) return hipSuccess;
    const long long units = (long long)p.row_blocks * p.splits, grid = (units + 7) / 8 * 8 * p.col_blocks;
    hipLaunchKernelGGL((head_range_kernel<SH, EL>), dim3((unsigned)grid), dim3(64 * kTileWaves), SH::LDS_BYTES, stream, p);
    return hipGetLastError();
  });
}
hipError_t launch_head_ranges(const HeadRangeParams& p, bool f32, hipStream_t stream) {
  return f32 ? launch_type<TileF32>(p, stream) : launch_type<TileBf16>(p, stream);
}

template <typename EL>
static hipError_t allow_lds(bool dma, bool aligned) {
  return each_shape(dma, aligned, [](auto shape) {
    using SH = decltype(shape);
    return hipFuncSetAttribute((const void*)head_range_kernel<SH, EL>, hipFuncAttributeMaxDynamicSharedMemorySize, SH::LDS_BYTES);
  });
}
hipError_t prepare_head_ranges() {
  hipError_t e = hipSuccess;
  for (const int way : {0, 1, 2}) {
    if (e == hipSuccess) e = allow_lds<TileBf16>(way == 2, way == 1);
    if (e == hipSuccess) e = allow_lds<TileF32>(way == 2, way == 1);
  }
  return e;
}

}  // namespace ctcspec
