// draft_layer_forward: the transformer layer of the attention draft module (Sec. 3.1) - the base family's
// decoder layer (RMSNorm, rotary multi-head attention over the layer's own key/value cache, gated SiLU
// feed-forward, residuals) applied to the T draft positions of every sequence in parallel.
//
// The layer is four passes over its weight matrices (405 MB at the 7B shape) and one attention call; everything else
// is small.  A pass serves up to 64 columns (B*T) and runs in layer_tile_kernel; the kernel that follows it (rotary
// embedding, residual + norm, gate, residual) adds the partial sums of its k splits in a fixed order - same bits on
// every run.
#include <type_traits>
#include <utility>

#include "dma_tile.h"
#include "head_plan.h"
#include "layer_plan.h"

namespace ctcspec {

__device__ __forceinline__ unsigned short float_to_bf16_bits(float f) {
  unsigned int u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;  // NaN
  return (unsigned short)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// ---- a pass: the tile loop of the heads --------------------------------------------------------------------------
// The activations are fp32 values carried as two bf16 numbers (value = high + low, 16 bits of mantissa), so the products
// lose nothing to a rounding of the activations.  A workgroup = ROWS weight rows x all columns of the pass x one of `splits` ranges of k.  Tile columns come in groups of
// 32: the high parts of 16 columns, then their low parts, so that a wavefront holds both products of a column and
// leaves one sum per (column, row): part[split][column][row], added up by the kernel that follows in ascending order.
// Why this split: a pass is bound by what a compute unit takes in per step - its weight rows from HBM and all
// columns' activations from L2, about 45 GB/s together - so the rows of a workgroup and the number of splits are chosen
// to fill the 256 compute units in as few rounds as possible (layer_plan.h), not by the matrix alone.
// Measured at the 7B shape (passes over 101, 34, 180 and 90 MB), all four passes together: 8 columns 75 us = 5.4 TB/s,
// 64 columns 106 us (through registers, steps in order: 84 to 88 and 117).  Before that, wavefronts streamed 16-row units past activations held in LDS, 16 columns at a time: 107 us
// for 8 columns (three accumulators per wavefront for ranges that cross row tiles, 6 MB of partial tiles per pass),
// 16 passes of 28 to 32 us for 64.
struct LayerTileParams {
  const void* w;      // [N][K] bf16
  const void* x;      // [2][plane_cols][K] bf16, the pass's columns from col0 on
  const void* zeros;
  float* part;        // [splits][cols][N]
  int N, K, cols, plane_cols, col0, row_blocks, splits;
  bool streamed;      // streamed_weights (head_plan.h), by the whole layer
  int trips, more;    // k trips of a split; the first `more` splits have one more
};
struct LayerColumns {
  int cols, plane_cols;
  __device__ __forceinline__ int operator()(int r) const {
    const int col = (r >> 5) * 16 + (r & 15);
    return ((r >> 4) & 1) * plane_cols + (col < cols ? col : cols - 1);
  }
  __device__ __forceinline__ int row_or_none(int r) const { return (r >> 5) * 16 + (r & 15) < cols ? (*this)(r) : -1; }
};
template <typename SH>
__global__ __launch_bounds__(64 * kTileWaves) void layer_tile_kernel(LayerTileParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  static_assert(kLtTripK * 2 % SH::STEPB == 0 && SH::CTW % 2 == 0, "whole steps, column tiles in high / low pairs");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave / SH::WC, wc = wave % SH::WC;
  const int c = lane & 15, g = lane >> 4;
  // (row block and split from the grid, the trips of a split without a division: those were a quarter of the way to the first load)
  const int rb = blockIdx.x, split = blockIdx.y;
  const int t0 = split * p.trips + (split < p.more ? split : p.more), t1 = t0 + p.trips + (split < p.more ? 1 : 0);
  GemmTileArgs t;
  t.w = (const unsigned char*)p.w + (size_t)t0 * kLtTripK * 2;
  t.hidden = (const unsigned char*)p.x + (size_t)p.col0 * p.K * 2 + (size_t)t0 * kLtTripK * 2;
  t.zeros = p.zeros; t.D = (t1 - t0) * kLtTripK; t.pitch = p.K; t.V = p.N; t.row_base = rb * SH::ROWS; t.streamed = p.streamed;
  f32x4 acc[SH::RT][SH::CTW];
  if constexpr (SH::DMA) dma_tile<SH, TileBf16>(t, LayerColumns{p.cols, p.plane_cols}, smem, acc);
  else gemm_tile<4, SH, TileBf16>(t, LayerColumns{p.cols, p.plane_cols}, smem, acc);
  float* out = p.part + (size_t)split * p.cols * p.N;
#pragma unroll
  for (int ct = 0; ct < SH::CTW; ct += 2) {
    const int col = wc * 8 * SH::CTW + ct * 8 + c;
    if (col >= p.cols) continue;
#pragma unroll
    for (int rt = 0; rt < SH::RT; ++rt) {
      const int row = t.row_base + (wr * SH::RT + rt) * 16 + g * 4;
      if (row < p.N) *(f32x4*)(out + (size_t)col * p.N + row) = acc[rt][ct] + acc[rt][ct + 1];  // N: a multiple of 16
    }
  }
}

// Entry (col, row) of the product: the splits' sums in ascending order.
__device__ __forceinline__ float pass_result(const float* __restrict__ part, const LayerPlan& pl, int col, int row) {
  const float* t = part + (size_t)col * pl.N + row;
  const size_t stride = (size_t)pl.cols * pl.N;
  float s = 0.f;
#pragma unroll 4
  for (int q = 0; q < pl.splits; ++q) s += t[q * stride];
  return s;
}

// fp32 value -> two bf16 numbers whose sum carries 16 bits of its mantissa, at index i of a [2][plane] array
__device__ __forceinline__ void store_split(unsigned short* planes, size_t plane_elems, size_t i, float v) {
  const unsigned short hi = float_to_bf16_bits(v);
  planes[i] = hi;
  planes[plane_elems + i] = float_to_bf16_bits(v - bf16_bits_to_float(hi));
}

__device__ __forceinline__ float block_sum_256(float v, float* red) {
  v = wave_sum_f32(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// The input of the first pass: x * gain as two bf16 numbers (the product of two bf16 numbers is exact in 16 mantissa
// bits) and the sums of x^2 over each 256 elements.  One block per (column, 256 elements).
__global__ __launch_bounds__(256) void dl_scale_in_kernel(const unsigned short* __restrict__ x,
                                                          const unsigned short* __restrict__ gain, unsigned short* planes,
                                                          float* ss, int BT, int D) {
  __shared__ float red[4];
  const int nseg = D / 256, col = blockIdx.x / nseg, seg = blockIdx.x - col * nseg, d = seg * 256 + threadIdx.x;
  const float v = bf16_bits_to_float(x[(size_t)col * D + d]);
  store_split(planes, (size_t)BT * D, (size_t)col * D + d, v * bf16_bits_to_float(gain[d]));
  const float t = block_sum_256(v * v, red);
  if (threadIdx.x == 0) ss[col * nseg + seg] = t;
}

struct LayerParams {
  const unsigned short* x;     // [B*T][D] bf16 input hidden states
  const unsigned short* ln1;   // [D]
  const unsigned short* ln2;   // [D]
  const int32_t* pos0;         // [B]
  int B, T, D, H, dh, F;
  float eps, log2_theta;
  // workspace
  // activations that feed a matrix product are [2][B*T][K] bf16: high parts, then low parts
  unsigned short* q;           // [B][H][T][dh]
  unsigned short* arows;       // [2][B*T][D] attention output, heads side by side
  float* h1;                   // [B*T][D] residual stream after attention
  unsigned short* xn2;         // [2][B*T][D]
  unsigned short* act;         // [2][B*T][F]
  int32_t* n_rows;             // [B] = T
  unsigned long long* causal;  // [B][T] bit j of row t set for j <= t
  float* ss1;                  // [B*T][D/256] partial sums of x^2
  float* ss2;                  // [B*T][D/256] partial sums of h1^2
  // outputs
  unsigned short* k_new;       // [B][H][T][dh]
  unsigned short* v_new;       // [B][H][T][dh]
  unsigned short* out;         // [B*T][D]
  float* out_f32;              // [B*T][D] or null
  const float* part;
  int col0, cols;              // columns of the current pass
};

// RMSNorm is a per-column scalar times an elementwise gain, and the scalar commutes with the matrix product
// that follows: the product is taken of x * gain, the kernel that consumes it multiplies by
// 1 / sqrt(mean(x^2) + eps).  The sum of squares is left as one partial sum per 256 elements, added up by the
// consumer in ascending order.
__device__ __forceinline__ float inv_rms(const float* __restrict__ ss, int col, int nseg, int D, float eps) {
  float t = 0.f;
  for (int i = 0; i < nseg; ++i) t += ss[col * nseg + i];
  return 1.0f / sqrtf(t / (float)D + eps);
}

// q, k, v of the pass's columns: sum of the partial tiles times the norm's scalar (the first pass took x * gain and
// left the sums of x^2), rotary embedding on q and k, bf16, head-major layout
__global__ __launch_bounds__(256) void dl_qkv_finish_kernel(LayerParams p, LayerPlan pl) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && p.col0 == 0) {
    // the row counts and the causal mask that the attention call takes
    for (int i = threadIdx.x; i < p.B; i += 256) p.n_rows[i] = p.T;
    for (int i = threadIdx.x; i < p.B * p.T; i += 256) {
      const int t = i % p.T;
      p.causal[i] = t >= 63 ? ~0ull : ((2ull << t) - 1ull);
    }
  }
  // grid: (blocks over the column's 3 H dh / 2 pairs, column of the pass) - no division by a runtime number per
  // element except the one that finds the head
  const int half = p.dh / 2;
  const int per_col = 3 * p.H * half;
  const int cl = blockIdx.y, col = p.col0 + cl, b = col / p.T, t = col - b * p.T;
  const float inv = inv_rms(p.ss1, col, p.D / 256, p.D, p.eps);
  for (int rem = blockIdx.x * 256 + threadIdx.x; rem < per_col; rem += gridDim.x * 256) {
    const int hq = rem / half, i = rem - hq * half;  // hq: 0..H-1 q heads, H..2H-1 k heads, 2H..3H-1 v heads
    const int row = hq * p.dh + i;
    float a = inv * pass_result(p.part, pl, cl, row), c = inv * pass_result(p.part, pl, cl, row + half);
    const int kind = hq / p.H, h = hq - kind * p.H;
    if (kind < 2) {
      // pair (i, i + dh/2) turned by the angle pos * theta^(-2i/dh)
      const float ang = (float)(p.pos0[b] + t) * exp2f(-2.0f * (float)i / (float)p.dh * p.log2_theta);
      float sn, cs;
      sincosf(ang, &sn, &cs);
      const float ra = a * cs - c * sn, rc = c * cs + a * sn;
      a = ra;
      c = rc;
    }
    unsigned short* dst = (kind == 0 ? p.q : kind == 1 ? p.k_new : p.v_new) + (((size_t)b * p.H + h) * p.T + t) * p.dh;
    dst[i] = float_to_bf16_bits(a);
    dst[i + half] = float_to_bf16_bits(c);
  }
}

// h1 = x + attention projection; h1 * ln2 (as two bf16 numbers) and the partial sums of h1^2.
// One block per (column of the pass, 256 elements).
__global__ __launch_bounds__(256) void dl_oproj_finish_kernel(LayerParams p, LayerPlan pl) {
  __shared__ float red[4];
  const int nseg = p.D / 256;
  const int cl = blockIdx.x / nseg, seg = blockIdx.x - cl * nseg, tid = threadIdx.x;
  const int col = p.col0 + cl, d = seg * 256 + tid;
  const size_t o = (size_t)col * p.D + d;
  const float v = bf16_bits_to_float(p.x[o]) + pass_result(p.part, pl, cl, d);
  p.h1[o] = v;
  store_split(p.xn2, (size_t)p.B * p.T * p.D, o, v * bf16_bits_to_float(p.ln2[d]));
  const float ss = block_sum_256(v * v, red);
  if (tid == 0) p.ss2[col * nseg + seg] = ss;
}

// act = silu(gate) * up; rows [0, F) of the fused matrix are the gate, rows [F, 2F) the up projection.  Four elements a
// thread: with one, 64 columns of 11008 are 2752 workgroups of single loads, 8.2 us against 6.2.  (The other kernels
// between the passes are smaller; four elements a thread made a layer of 1024 4 % slower: fewer wavefronts wait longer.)
__global__ __launch_bounds__(256) void dl_gate_finish_kernel(LayerParams p, LayerPlan pl) {
  typedef __attribute__((ext_vector_type(4))) unsigned short u16x4;
  const int cl = blockIdx.y;  // grid: (blocks over F / 4, column of the pass)
  const size_t plane = (size_t)p.B * p.T * p.F, stride = (size_t)pl.cols * pl.N;
  for (int f = 4 * (blockIdx.x * 256 + threadIdx.x); f < p.F; f += 4 * gridDim.x * 256) {
    const float* t = p.part + (size_t)cl * pl.N + f;
    f32x4 sg = {0.f, 0.f, 0.f, 0.f}, su = sg;
#pragma unroll 4
    for (int q = 0; q < pl.splits; ++q) {  // ascending, as pass_result
      sg += *(const f32x4*)(t + q * stride);
      su += *(const f32x4*)(t + q * stride + p.F);
    }
    const float inv = inv_rms(p.ss2, p.col0 + cl, p.D / 256, p.D, p.eps);
    u16x4 hi, lo;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float gt = inv * sg[e], up = inv * su[e], v = gt / (1.0f + expf(-gt)) * up;
      hi[e] = float_to_bf16_bits(v);
      lo[e] = float_to_bf16_bits(v - bf16_bits_to_float(hi[e]));
    }
    const size_t at = (size_t)(p.col0 + cl) * p.F + f;
    *(u16x4*)(p.act + at) = hi;
    *(u16x4*)(p.act + plane + at) = lo;
  }
}

// out = h1 + feed-forward output
__global__ __launch_bounds__(256) void dl_down_finish_kernel(LayerParams p, LayerPlan pl) {
  const int cl = blockIdx.y;  // grid: (blocks over D, column of the pass)
  for (int d = blockIdx.x * 256 + threadIdx.x; d < p.D; d += gridDim.x * 256) {
    const size_t o = (size_t)(p.col0 + cl) * p.D + d;
    const float v = p.h1[o] + pass_result(p.part, pl, cl, d);
    if (p.out_f32) p.out_f32[o] = v;
    p.out[o] = float_to_bf16_bits(v);
  }
}

// ---- host side ---------------------------------------------------------------------------------------------------
static int device_cus() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
      cus = n;
    else
      cus = 256;
  }
  return cus;
}

// rows x 16, 32 or 64 columns (twice as many tile columns); which one: layer_plan.h
using LayerTile128x16 = DmaShape<8, 1, 2, 256, 4, 3>;
using LayerTileShort = TileShape<8, 2, 128, 1, true, true>;  // through registers (layer_plan.h: through_registers)
using LayerTile256x16 = DmaShape<8, 2, 2, 128, 4, 4>;
using LayerTile128x32 = DmaShape<4, 2, 2, 256, 3, 3>;
using LayerTile192x32 = DmaShape<4, 3, 2, 128, 4, 4>;
using LayerTile256x32 = DmaShape<4, 4, 2, 128, 4, 4>;
using LayerTile128x64 = DmaShape<4, 2, 4, 256, 3, 2>;
using LayerTile192x64 = DmaShape<4, 3, 4, 128, 4, 4>;
using LayerTile256x64 = DmaShape<4, 4, 4, 128, 3, 3>;
template <typename SH>
static hipError_t launch_shape(const LayerTileParams& tp, hipStream_t stream) {
  hipLaunchKernelGGL(layer_tile_kernel<SH>, dim3((unsigned)tp.row_blocks, (unsigned)tp.splits), dim3(64 * kTileWaves), SH::LDS_BYTES,
                     stream, tp);
  return hipGetLastError();
}
static hipError_t launch_pass(LayerTileParams& tp, const LayerPlan& plan, hipStream_t stream) {
  const int rows = plan.rows;
  tp.row_blocks = (tp.N + rows - 1) / rows;
  tp.trips = tp.K / kLtTripK / tp.splits;
  tp.more = tp.K / kLtTripK % tp.splits;
  if (through_registers(plan, tp.streamed)) return launch_shape<LayerTileShort>(tp, stream);
  switch (tile_columns(tp.cols)) {
    case 32: return rows == 128 ? launch_shape<LayerTile128x16>(tp, stream) : launch_shape<LayerTile256x16>(tp, stream);
    case 64:
      if (rows == 128) return launch_shape<LayerTile128x32>(tp, stream);
      return rows == 192 ? launch_shape<LayerTile192x32>(tp, stream) : launch_shape<LayerTile256x32>(tp, stream);
    default:
      if (rows == 128) return launch_shape<LayerTile128x64>(tp, stream);
      return rows == 192 ? launch_shape<LayerTile192x64>(tp, stream) : launch_shape<LayerTile256x64>(tp, stream);
  }
}

template <typename... SH>
static hipError_t allow_lds() {
  hipError_t e = hipSuccess;
  ((e = e == hipSuccess ? hipFuncSetAttribute((const void*)layer_tile_kernel<SH>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                              SH::LDS_BYTES)
                        : e),
   ...);
  return e;
}
hipError_t prepare_draft_layer() {
  return allow_lds<LayerTileShort, LayerTile128x16, LayerTile256x16, LayerTile128x32, LayerTile192x32, LayerTile256x32, LayerTile128x64,
                   LayerTile192x64, LayerTile256x64>();
}

}  // namespace ctcspec

using namespace ctcspec;

extern "C" size_t draft_layer_workspace_bytes(int B, int T, int D, int H, int F) {
  if (B < 1 || T < 1 || D < 1 || H < 1 || F < 1) return 0;
  return layer_workspace(B, T, D, H, F, device_cus(), true).total;
}

extern "C" int draft_layer_forward(ctcspec_ctx* ctx, ctcspec_dtype dt, const void* x,
                                   const ctcspec_layer_weights* w, const int32_t* pos0, void* k_cache,
                                   void* v_cache, const int64_t* kv_off, const int32_t* ctx_len, int kv_cap, int B,
                                   int T, int D, int H, int F, float rms_eps, float rope_theta, void* workspace,
                                   size_t workspace_bytes, void* q_out, void* k_new, void* v_new, void* out, float* out_f32) {
  if (!ctx) return CTCSPEC_EINVAL;
  if (const int owed = flush_deferred(ctx)) return owed;
  CTCSPEC_REQUIRE(ctx, x && w && pos0 && k_cache && v_cache && kv_off && ctx_len && workspace && k_new && v_new && out,
                  CTCSPEC_EINVAL, "draft_layer_forward: null pointer");
  CTCSPEC_REQUIRE(ctx, w->ln1 && w->wqkv && w->wo && w->ln2 && w->wgu && w->wd, CTCSPEC_EINVAL,
                  "draft_layer_forward: null weight pointer");
  CTCSPEC_REQUIRE(ctx, dt == CTCSPEC_BF16, CTCSPEC_EUNSUPPORTED, "draft_layer_forward: bf16 only");
  CTCSPEC_REQUIRE(ctx, B > 0 && T > 0 && D > 0 && H > 0 && F > 0 && kv_cap >= 0, CTCSPEC_EINVAL,
                  "draft_layer_forward: sizes must be positive");
  CTCSPEC_REQUIRE(ctx, D % H == 0 && D % 256 == 0 && F % 256 == 0 && (D / H) % 8 == 0 && D / H <= CTCSPEC_MAX_HEAD_DIM,
                  CTCSPEC_EUNSUPPORTED,
                  "draft_layer_forward: D and F must be multiples of 256, D/H a multiple of 8 and <= %d",
                  CTCSPEC_MAX_HEAD_DIM);
  CTCSPEC_REQUIRE(ctx, T <= 64 && T <= ctx->lim.max_nodes && B <= ctx->lim.max_batch && H <= ctx->lim.max_heads &&
                           D / H <= ctx->lim.max_head_dim,
                  CTCSPEC_EUNSUPPORTED, "draft_layer_forward: shape exceeds the context's limits");
  CTCSPEC_REQUIRE(ctx, rms_eps >= 0.f && rope_theta > 1.f, CTCSPEC_EINVAL, "draft_layer_forward: bad eps or theta");
  const void* ptrs[] = {x, w->ln1, w->wqkv, w->wo, w->wgu, w->wd, workspace, q_out, k_new, v_new, out, k_cache, v_cache};
  for (const void* q : ptrs)
    CTCSPEC_REQUIRE(ctx, aligned16(q), CTCSPEC_EINVAL, "draft_layer_forward: pointers must be 16-byte aligned");
  const int cus = device_cus();
  const LayerWorkspace lw = layer_workspace(B, T, D, H, F, cus, false);
  CTCSPEC_REQUIRE(ctx, workspace_bytes >= lw.total, CTCSPEC_EINVAL,
                  "draft_layer_forward: workspace of %zu bytes needed, %zu given", lw.total, workspace_bytes);

  unsigned char* ws = (unsigned char*)workspace;
  LayerParams p;
  p.x = (const unsigned short*)x; p.ln1 = (const unsigned short*)w->ln1; p.ln2 = (const unsigned short*)w->ln2;
  p.pos0 = pos0; p.B = B; p.T = T; p.D = D; p.H = H; p.dh = D / H; p.F = F;
  p.eps = rms_eps; p.log2_theta = log2f(rope_theta);
  p.q = q_out ? (unsigned short*)q_out : (unsigned short*)(ws + lw.q);
  p.arows = (unsigned short*)(ws + lw.arows); p.h1 = (float*)(ws + lw.h1); p.xn2 = (unsigned short*)(ws + lw.xn2);
  p.act = (unsigned short*)(ws + lw.act); p.n_rows = (int32_t*)(ws + lw.n_rows);
  p.causal = (unsigned long long*)(ws + lw.causal); p.ss1 = (float*)(ws + lw.ss1); p.ss2 = (float*)(ws + lw.ss2);
  p.k_new = (unsigned short*)k_new; p.v_new = (unsigned short*)v_new; p.out = (unsigned short*)out; p.out_f32 = out_f32;
  p.part = (const float*)(ws + lw.part); p.col0 = 0; p.cols = 0;
  const int BT = B * T;
  hipStream_t st = ctx->stream;

  // one pass over a weight matrix per block of 64 columns, each followed by the kernel that consumes its sums
  auto gemm_passes = [&](const void* wmat, int N, int K, const unsigned short* xin, auto&& finish) -> int {
    for (int col0 = 0; col0 < BT; col0 += kLtMaxCols) {
      LayerPlan plan;
      p.col0 = col0;
      p.cols = BT - col0 < kLtMaxCols ? BT - col0 : kLtMaxCols;
      CTCSPEC_REQUIRE(ctx, make_plan(plan, N, K, p.cols, BT, cus), CTCSPEC_EUNSUPPORTED,
                      "draft_layer_forward: a %d x %d matrix does not fit the tile kernel", N, K);
      LayerTileParams tp;
      tp.streamed = streamed_weights(2LL * (4LL * D * D + 3LL * D * F), 2LL * K);
      tp.w = wmat; tp.x = xin; tp.zeros = ctx->zeros; tp.part = (float*)(ws + lw.part);
      tp.N = N; tp.K = K; tp.cols = p.cols; tp.plane_cols = BT; tp.col0 = col0; tp.splits = plan.splits;
      CTCSPEC_HIP(ctx, launch_pass(tp, plan, st));
      finish(plan);
      CTCSPEC_HIP(ctx, hipGetLastError());
    }
    return CTCSPEC_OK;
  };
  auto blocks_for = [](long long n) { long long b = (n + 255) / 256; return (unsigned)(b > 1024 ? 1024 : (b < 1 ? 1 : b)); };

  // (the scaled input takes the place of the second norm's, which is written after the first pass)
  hipLaunchKernelGGL(dl_scale_in_kernel, dim3((unsigned)(BT * (D / 256))), dim3(256), 0, st, p.x, p.ln1, p.xn2, p.ss1, BT, D);
  CTCSPEC_HIP(ctx, hipGetLastError());
  int rc = gemm_passes(w->wqkv, 3 * D, D, p.xn2, [&](const LayerPlan& pl) {
    hipLaunchKernelGGL(dl_qkv_finish_kernel, dim3(blocks_for((long long)3 * H * (p.dh / 2)), p.cols), dim3(256), 0, st, p, pl);
  });
  if (rc != CTCSPEC_OK) return rc;
  rc = tree_verify_attn_rows(ctx, dt, p.q, k_cache, v_cache, kv_off, ctx_len, kv_cap, k_new, v_new, p.n_rows,
                             (const uint64_t*)p.causal, B, H, p.dh, T, 1.0f / sqrtf((float)p.dh), nullptr, p.arows,
                             (long long)BT * D, 2LL * (4LL * D * D + 3LL * D * F));
  if (rc != CTCSPEC_OK) return rc;
  rc = gemm_passes(w->wo, D, D, p.arows, [&](const LayerPlan& pl) {
    hipLaunchKernelGGL(dl_oproj_finish_kernel, dim3(p.cols * (D / 256)), dim3(256), 0, st, p, pl);
  });
  if (rc != CTCSPEC_OK) return rc;
  rc = gemm_passes(w->wgu, 2 * F, D, p.xn2, [&](const LayerPlan& pl) {
    hipLaunchKernelGGL(dl_gate_finish_kernel, dim3(blocks_for((long long)F / 4), p.cols), dim3(256), 0, st, p, pl);
  });
  if (rc != CTCSPEC_OK) return rc;
  rc = gemm_passes(w->wd, D, F, p.act, [&](const LayerPlan& pl) {
    hipLaunchKernelGGL(dl_down_finish_kernel, dim3(blocks_for((long long)D), p.cols), dim3(256), 0, st, p, pl);
  });
  return rc;
}
