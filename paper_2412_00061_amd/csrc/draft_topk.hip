// ctc_draft_topk: LM head over vocabulary + blank, log-softmax and per-slot top-k in one pass over W.
//
// The head weights are read exactly once.  A workgroup owns 128 consecutive vocabulary rows; it
// leaves, per column (= draft slot of some sequence), the running max, the sum of exponentials and
// its k best (logit, id) pairs.  A second, tiny kernel merges the partials of all workgroups into
// lse / topk_id / topk_logp.  (Merging inside the first kernel behind an atomic ticket needs a
// device-scope release fence in every workgroup; on this GPU that is an L2 write-back per workgroup
// and costs far more than the launch of a second kernel.)
//
// Two producers of the 128 x columns logit block exist:
//   * lmhead_bf16_mfma_kernel  - bf16 operands, v_mfma_f32_16x16x32_bf16, HBM-streaming design: a wavefront
//                                streams 16 rows, the hidden states of all columns sit in LDS (up to 11
//                                columns at D = 4096)
//   * lmhead_tile_kernel       - everything else (more columns, other hidden sizes, float operands): the tile
//                                loop of dma_tile.h (rows that start anywhere, single steps and single row
//                                blocks: gemm_tile.h), both operands stepping through LDS
// Both hand the block over in LDS to the same epilogue.  Vocabularies that do not fill the chip are cut along the hidden
// dimension as well (head_ranges.h); lmhead_columns_kernel then finishes a column.
#include <mutex>
#include <type_traits>
#include <utility>

#include <hip/hip_ext.h>

#include "dma_tile.h"
#include "head_ranges.h"
#include "topk_merge.h"

namespace ctcspec {

constexpr int kZStride = kRowsPerBlock + 4;  // floats per column in the LDS logit block
struct LmHeadParams {
  const void* hidden;
  const void* w;
  const float* bias;
  int BT, D, Vp1, k;
  int KC;        // mfma kernel: hidden elements per column held in LDS (= D)
  int hs_bytes;  // mfma kernel: bytes of the LDS hidden-state region
  unsigned int hs_magic;  // mfma kernel: ceil(2^32 / (KC / 8)), for index / (KC / 8) by multiplication
  int n_blocks;
  const void* zeros;  // tile kernel: 256 bytes of zeros
  float* pmax;              // [kMaxCols][pstride]
  float* psum;              // [kMaxCols][pstride]
  unsigned long long* pkey; // [kMaxCols][kMaxTopk][pstride]
  int pstride;              // workgroups the partial arrays have room for
  int32_t* topk_id;
  float* topk_logp;
  float* lse;
  float* logits_out;
  bool streamed;      // streamed_weights (head_plan.h)
};

// What a vocabulary of a single row block leaves itself, to the bits of the merge kernel: 101 rows of 64 float, 4 columns 6.6 -> 4.1 us
// a call.
__device__ __forceinline__ float block_lse(float mx, float s) { return (mx > -INFINITY ? mx : -INFINITY) + __logf(s); }
__device__ __forceinline__ void store_ranked(const LmHeadParams& p, int col, int r, unsigned long long key, float lse) {
  p.topk_id[col * p.k + r] = (int32_t)rank_key_index(key);
  p.topk_logp[col * p.k + r] = rank_key_value(key) - lse;
}

// Epilogue shared by both producers.  zbuf holds the block's logits column-major:
// zbuf[col * kZStride + r] = z of row (blockIdx.x*128 + r), -inf for rows >= Vp1.
// Whole wavefronts must call this (the reductions use every lane).
// ALONE: the only row block, which has nothing to merge.  (As a branch per column and rank it cost the others: 64 columns x 12406 rows of 512,
// k = 7, 27.5 -> 29.3 us, 21 columns, k = 4, 12.5 -> 13.0.)
template <bool ALONE>
__device__ __forceinline__ void lmhead_block_epilogue(const LmHeadParams& p, const float* zbuf) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nwaves = blockDim.x >> 6;
  const int row_base = blockIdx.x * kRowsPerBlock;
  const int k = p.k;

  if (p.logits_out) {
    for (int idx = tid; idx < p.BT * kRowsPerBlock; idx += blockDim.x) {
      int m = idx / kRowsPerBlock, r = idx % kRowsPerBlock;
      if (row_base + r < p.Vp1) p.logits_out[(size_t)m * p.Vp1 + row_base + r] = zbuf[m * kZStride + r];
    }
  }

  // per column: max, sum of exponentials, k best keys of this block's 128 rows
  for (int m = wave; m < p.BT; m += nwaves) {
    float z0 = zbuf[m * kZStride + lane];
    float z1 = zbuf[m * kZStride + lane + 64];
    int id0 = row_base + lane, id1 = row_base + lane + 64;
    float mx = wave_max_f32(fmaxf(z0, z1));
    float e = 0.f;
    if (mx > -INFINITY) e = __expf(z0 - mx) + __expf(z1 - mx);
    float s = wave_sum_f32(e);
    unsigned long long a = id0 < p.Vp1 ? rank_key(z0, (unsigned)id0) : 0ull;
    unsigned long long b = id1 < p.Vp1 ? rank_key(z1, (unsigned)id1) : 0ull;
    if (b > a) { unsigned long long t = a; a = b; b = t; }
    const size_t slot = (size_t)m * p.pstride + blockIdx.x;
    const float lse = ALONE ? block_lse(mx, s) : 0.f;
    for (int r = 0; r < k; ++r) {
      unsigned long long best = wave_max_u64(a);
      if (lane == 0) {
        if constexpr (ALONE) store_ranked(p, m, r, best, lse);
        else p.pkey[((size_t)m * kMaxTopk + r) * p.pstride + blockIdx.x] = best;
      }
      if (a == best) { a = b; b = 0ull; }
    }
    if (lane == 0) {
      if constexpr (!ALONE) { p.pmax[slot] = mx; p.psum[slot] = s; }
      else if (p.lse) p.lse[m] = lse;
    }
  }
}

// The same epilogue for many columns: a lane per column instead of a wavefront per column.  Wavefront w scans
// rows 16w .. 16w+15 of every column (lane = column): groups of KMAX keys are sorted and merged, the k best stay, sorted, in
// registers.  The eight wavefronts' (max, sum, keys) of a column are joined in three rounds through LDS, half of the
// wavefronts handing theirs to the other half.  `part` is LDS behind zbuf: 4 x kMaxCols x (2 floats + KMAX keys).
// Bound: instruction issue of single wavefronts.  With sorted insertion of every key and the first wavefront joining all
// eight lists that way: 40 columns x 41675 rows of 3840, k = 6, 107 us a call,
// 88.5 so; 64 columns x 32001 of 4096, k = 4, 64.9 to 65.3 / 60.6 to 63.6 (by card and placement).
template <int KMAX>
__device__ __forceinline__ void lmhead_block_epilogue_wide(const LmHeadParams& p, const float* zbuf, unsigned char* part) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row_base = blockIdx.x * kRowsPerBlock;
  static_assert(kMaxCols == 64 && kRowsPerBlock == 16 * kMfmaWaves && kMfmaWaves == 8, "a lane per column - every lane writes to `part` -, sixteen rows per wavefront");
  if (p.logits_out) {
    for (int idx = tid; idx < p.BT * kRowsPerBlock; idx += blockDim.x) {
      int m = idx / kRowsPerBlock, r = idx % kRowsPerBlock;
      if (row_base + r < p.Vp1) p.logits_out[(size_t)m * p.Vp1 + row_base + r] = zbuf[m * kZStride + r];
    }
  }
  constexpr int HANDED = kMfmaWaves / 2;
  float* pm = (float*)part;                                                        // [HANDED][kMaxCols]
  float* ps = pm + HANDED * kMaxCols;                                              // [HANDED][kMaxCols]
  unsigned long long* pk = (unsigned long long*)(ps + HANDED * kMaxCols);          // [HANDED][KMAX][kMaxCols]
  const int m = lane < p.BT ? lane : p.BT - 1;  // (lanes without a column repeat the last one's and write nothing)
  f32x4 z[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) z[q] = *(const f32x4*)(zbuf + m * kZStride + 16 * wave + 4 * q);
  float mx = -INFINITY;
#pragma unroll
  for (int q = 0; q < 4; ++q) mx = fmaxf(mx, fmaxf(fmaxf(z[q][0], z[q][1]), fmaxf(z[q][2], z[q][3])));
  float sum = 0.f;
  unsigned long long keys[16 / KMAX][KMAX];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int id = row_base + 16 * wave + 4 * q + i;
      if (mx > -INFINITY) sum += __expf(z[q][i] - mx);
      keys[(4 * q + i) / KMAX][(4 * q + i) % KMAX] = id < p.Vp1 ? rank_key(z[q][i], (unsigned)id) : 0ull;
    }
#pragma unroll
  for (int g = 0; g < 16 / KMAX; ++g) sort_keys<KMAX>(keys[g]);
#pragma unroll
  for (int step = 1; step < 16 / KMAX; step *= 2)
#pragma unroll
    for (int g = 0; g + step < 16 / KMAX; g += 2 * step) merge_sorted_lists<KMAX>(keys[g], keys[g + step]);
#pragma unroll
  for (int half = HANDED; half >= 1; half /= 2) {
    if (wave >= half && wave < 2 * half) {
      const int at = (wave - half) * kMaxCols + lane;
      pm[at] = mx;
      ps[at] = sum;
#pragma unroll
      for (int r = 0; r < KMAX; ++r) pk[((wave - half) * KMAX + r) * kMaxCols + lane] = keys[0][r];
    }
    lds_barrier();  // (the logits' stores stay in flight)
    if (wave < half) {
      const float om = pm[wave * kMaxCols + lane], osum = ps[wave * kMaxCols + lane];
      const float mn = fmaxf(mx, om);
      if (mn > -INFINITY) sum = (mx > -INFINITY ? sum * __expf(mx - mn) : 0.f) + (om > -INFINITY ? osum * __expf(om - mn) : 0.f);
      mx = mn;
      unsigned long long other[KMAX];
#pragma unroll
      for (int r = 0; r < KMAX; ++r) other[r] = pk[(wave * KMAX + r) * kMaxCols + lane];
      merge_sorted_lists<KMAX>(keys[0], other);
    }
    if (half > 1) lds_barrier();  // read before the next round overwrites it
  }
  if (wave == 0 && lane < p.BT && p.n_blocks == 1) {
    const float lse = block_lse(mx, sum);
    if (p.lse) p.lse[lane] = lse;
#pragma unroll
    for (int r = 0; r < KMAX; ++r)
      if (r < p.k) store_ranked(p, lane, r, keys[0][r], lse);
  } else if (wave == 0 && lane < p.BT) {
    const size_t slot = (size_t)lane * p.pstride + blockIdx.x;
    p.pmax[slot] = mx;
    p.psum[slot] = sum;
#pragma unroll
    for (int r = 0; r < KMAX; ++r)
      if (r < p.k) p.pkey[((size_t)lane * kMaxTopk + r) * p.pstride + blockIdx.x] = keys[0][r];
  }
}

// Merge of the per-workgroup partials: one wavefront per column (the merge itself: topk_merge.h).
template <int KMAX>
__global__ __launch_bounds__(64) void lmhead_merge_kernel(LmHeadParams p) {
  const int lane = threadIdx.x, k = p.k;
  const int col[1] = {(int)blockIdx.x};
  float lse[1];
  unsigned long long best[1][KMAX];
  merge_topk_columns<KMAX, 1>(p.pmax, p.psum, p.pkey, p.pstride, p.n_blocks, k, col, lse, best);
  if (lane == 0 && p.lse) p.lse[col[0]] = lse[0];
  if (lane < k) {
    unsigned long long key = 0ull;
#pragma unroll
    for (int r = 0; r < KMAX; ++r) key = lane == r ? best[0][r] : key;
    p.topk_id[col[0] * k + lane] = (int32_t)rank_key_index(key);
    p.topk_logp[col[0] * k + lane] = rank_key_value(key) - lse[0];
  }
}

// A column in one workgroup: the ranges' sums, the bias, the logits' row, log-sum-exp and the k best keys (a lane's own,
// kept sorted, then the wavefront's off the heads of the lanes' lists, then the workgroup's).
// Bound: latency - one round of loads, then the wavefronts' maxima; k insertions per row instead of only where the lanes'
// maxima leave candidates took the longer the more rows a thread holds.
template <int KMAX, int NV>
__global__ __launch_bounds__(kHeadColumnThreads) void lmhead_columns_kernel(HeadRangeParams h, LmHeadParams p) {
  constexpr int WAVES = kHeadColumnThreads / 64;
  static_assert(WAVES * KMAX <= 64, "a lane per key in the last step");
  __shared__ float red[2 * WAVES];
  __shared__ unsigned long long keys[WAVES * KMAX];
  const int col = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  f32x4 z[NV];
  load_head_column<NV>(h, col, z);
  float mx = -INFINITY;
  KeyList<KMAX> list;
  list.clear();
#pragma unroll
  for (int j = 0; j < NV; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 4 * (j * kHeadColumnThreads + tid) + i;
      z[j][i] = row < p.Vp1 ? z[j][i] + (p.bias ? p.bias[row] : 0.f) : -INFINITY;
      mx = fmaxf(mx, z[j][i]);
    }
  if (p.logits_out) store_head_column<NV>(p.logits_out + (size_t)col * p.Vp1, p.Vp1, z);
  // k lanes have something at least as large as the k-th largest of the lanes' maxima: the rest is no candidate
  float left = mx, floor = -INFINITY;
  for (int r = 0; r < p.k; ++r) {
    floor = wave_max_f32(left);
    left = left == floor ? -INFINITY : left;
  }
  mx = wave_max_f32(mx);
#pragma unroll
  for (int j = 0; j < NV; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 4 * (j * kHeadColumnThreads + tid) + i;
      if (!(z[j][i] < floor) && row < p.Vp1) list.insert(rank_key(z[j][i], (unsigned)row));  // (not a number: a candidate)
    }
  if (lane == 0) red[wave] = mx;
#pragma unroll
  for (int r = 0; r < KMAX; ++r) {
    const unsigned long long best = wave_max_u64(list.v[0]);
    if (list.v[0] == best) list.pop();  // keys are distinct: one lane, or lanes that have none left
    if (lane == 0) keys[wave * KMAX + r] = best;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < WAVES; ++w) mx = fmaxf(mx, red[w]);
  float sum = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) sum += mx > -INFINITY ? __expf(z[j][i] - mx) : 0.f;
  sum = wave_sum_f32(sum);
  if (lane == 0) red[WAVES + wave] = sum;
  __syncthreads();
  if (wave != 0) return;
  sum = 0.f;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) sum += red[WAVES + w];
  const float lse = mx + __logf(sum);
  if (lane == 0 && p.lse) p.lse[col] = lse;
  unsigned long long mine = lane < WAVES * KMAX ? keys[lane] : 0ull, out = 0ull;
  for (int r = 0; r < p.k; ++r) {
    const unsigned long long best = wave_max_u64(mine);
    mine = mine == best ? 0ull : mine;
    out = lane == r ? best : out;
  }
  if (lane < p.k) {
    p.topk_id[col * p.k + lane] = (int32_t)rank_key_index(out);
    p.topk_logp[col * p.k + lane] = rank_key_value(out) - lse;
  }
}
template <int KMAX>
static hipError_t launch_columns(const HeadRangeParams& h, const LmHeadParams& p, hipStream_t stream) {
  return launch_for_rows(p.Vp1, [&](auto nv) {
    hipLaunchKernelGGL((lmhead_columns_kernel<KMAX, decltype(nv)::value>), dim3(p.BT), dim3(kHeadColumnThreads), 0, stream, h, p);
    return hipGetLastError();
  });
}

// ---- bf16 MFMA streaming producer -----------------------------------------------------------------
// 8 waves; wave w owns the 16 rows [block*128 + 16w, +16) over the whole hidden dimension.
// Per step of 256 hidden elements a wave issues 8 coalesced 16-byte loads (each instruction covers
// two rows x 512 contiguous bytes), parks them in its private LDS strip and reads them back in the
// MFMA A-operand layout (lane = row, 8 consecutive k).  Loads run STAGES-1 steps ahead in registers.
// The hidden states (the B operand) sit in LDS for the whole workgroup.
//
// Every global load of the streaming path is issued unconditionally and in a fixed number per step
// (rows past the vocabulary re-read its last row, the tail of the k loop is peeled instead of
// guarded): the waits can then name the exact number of younger loads that may stay in flight, and
// the prefetch pipeline never drains.  A load under a condition makes every later wait a full drain.
template <int NT, int STAGES>
__global__ __launch_bounds__(64 * kMfmaWaves) void lmhead_bf16_mfma_kernel(LmHeadParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  // a load instruction covers two rows x 512 bytes; within a row the lanes take the 16-byte chunks in an order
  // that lets the 16 lanes the LDS serves together (l .. l+7, l+16 .. l+23) write 256 consecutive bytes
  const int lrow = lane >> 5, lch = (lane & 7) | ((lane & 16) >> 1) | ((lane & 8) << 1);
  unsigned char* hs = smem;
  const int HSS = p.KC * 2 + 32;
  unsigned char* wst = smem + p.hs_bytes + wave * kWStageBytes;
  const int row0 = blockIdx.x * kRowsPerBlock + wave * 16;

  const unsigned char* wp[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    int row = row0 + 2 * j + lrow;
    row = row < p.Vp1 ? row : p.Vp1 - 1;  // the ragged last tile re-reads the last valid row
    wp[j] = (const unsigned char*)p.w + (size_t)row * p.D * 2 + lch * 16;
  }
  int bcol[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    int col = nt * 16 + c;
    bcol[nt] = (col < p.BT ? col : p.BT - 1) * HSS + g * 16;
  }

  f32x4 acc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int total_steps = p.D / 256;  // the host guarantees KC == D: the hidden states of all columns are in LDS

  // Hidden-state staging: every thread carries kHsPieces 16-byte pieces through registers (pieces past the
  // end repeat the last piece and are not written to LDS); they are requested before the first W loads.
  constexpr int kHsPieces = 12;
  const int per_row = p.KC / 8;  // 16-byte pieces per column
  const int hs_total = p.BT * per_row;
  u32x4 hreg[kHsPieces];
  int hs_dst[kHsPieces];  // LDS offset of piece u, -1: none
  size_t hs_src[kHsPieces];
#pragma unroll
  for (int u = 0; u < kHsPieces; ++u) {
    const int idx = tid + u * 64 * kMfmaWaves;
    const int cl = idx < hs_total ? idx : hs_total - 1;
    const int m = (int)__umulhi((unsigned)cl, p.hs_magic);  // cl / per_row
    const int q = cl - m * per_row;
    hs_dst[u] = idx < hs_total ? m * HSS + q * 16 : -1;
    hs_src[u] = (size_t)m * p.D * 2 + q * 16;
  }
  auto hs_request = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kHsPieces; ++u) hreg[u] = *(const u32x4*)((const unsigned char*)p.hidden + hs_src[u]);
  };
  auto hs_commit = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kHsPieces; ++u)
      if (hs_dst[u] >= 0) *(u32x4*)(hs + hs_dst[u]) = hreg[u];
  };

  // the order of the steps (step_segment in dma_tile.h): 8 columns of 4096 x 32001 rows take 3.3 us less so than in order
  struct Order {
    int seg, steps, place = 0, lap = 0;
    __device__ __forceinline__ int next() {
      const int now = place;
      place += seg;
      if (place >= steps) place = ++lap;
      return now;
    }
  };
  const int seg = step_segment((size_t)p.D * 2, 512);
  Order requested{seg, total_steps}, consumed{seg, total_steps};
  u32x4 v[STAGES][8];
  auto w_request = [&](auto stage_tag) __attribute__((always_inline)) {
    constexpr int ST = decltype(stage_tag)::value;
    const size_t at = (size_t)requested.next() * 512;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[ST][j] = __builtin_nontemporal_load((const u32x4*)(wp[j] + at));
    // keep the scheduler from mixing these loads with those of another step: the waits count loads in
    // issue order, and a stage whose loads are spread among younger ones can only be waited for late
    __builtin_amdgcn_sched_barrier(0);
  };
  // one step: W registers of stage ST -> LDS strip -> A fragments
  auto consume = [&](auto stage_tag) __attribute__((always_inline)) {
    constexpr int ST = decltype(stage_tag)::value;
    const int i = consumed.next();
#pragma unroll
    for (int j = 0; j < 8; ++j) *(u32x4*)(wst + (2 * j + lrow) * kWRowStride + lch * 16) = v[ST][j];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      bf16x8 a = __builtin_bit_cast(bf16x8, *(const u32x4*)(wst + c * kWRowStride + kk * 64 + g * 16));
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        bf16x8 b = __builtin_bit_cast(bf16x8, *(const u32x4*)(hs + bcol[nt] + (i * 256 + kk * 32) * 2));
        acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[nt], 0, 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto for_each_stage = [&](auto&& fn) __attribute__((always_inline)) {
    [&]<int... I>(std::integer_sequence<int, I...>) { (fn(std::integral_constant<int, I>{}), ...); }
    (std::make_integer_sequence<int, STAGES>{});
  };

  hs_request();
  for_each_stage([&](auto st) __attribute__((always_inline)) {
    if constexpr (decltype(st)::value < STAGES - 1) w_request(st);
  });

  {
    hs_commit();
    __syncthreads();
    // blocks of STAGES steps; step i refills, with step i + STAGES - 1, the stage that step i - 1 freed
    const int nblk = total_steps / STAGES;  // the host guarantees total_steps % STAGES == 0
    for (int blk = 0; blk + 1 < nblk; ++blk) {
      for_each_stage([&](auto st) __attribute__((always_inline)) {
        constexpr int SS = decltype(st)::value;
        w_request(std::integral_constant<int, (SS + STAGES - 1) % STAGES>{});
        consume(st);
      });
    }
    // last block: only its first step still has something to prefetch
    for_each_stage([&](auto st) __attribute__((always_inline)) {
      constexpr int SS = decltype(st)::value;
      if constexpr (SS == 0) w_request(std::integral_constant<int, STAGES - 1>{});
      consume(st);
    });
  }

  // hand the 128 x BT logit block to the epilogue (the W strips are no longer needed)
  __syncthreads();
  float* zbuf = (float*)(smem + p.hs_bytes);
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    int col = nt * 16 + c;
    if (col < p.BT) {
      f32x4 z;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        int row = row0 + g * 4 + i;
        z[i] = row < p.Vp1 ? acc[nt][i] + (p.bias ? p.bias[row] : 0.f) : -INFINITY;
      }
      *(f32x4*)(zbuf + col * kZStride + wave * 16 + g * 4) = z;
    }
  }
  __syncthreads();
  lmhead_block_epilogue<false>(p, zbuf);  // (a single row block takes another kernel)
}

// ---- tile producer: any hidden size and type --------------------------------------------------------------------
// The tile loop shared with the base-model head, 128 rows x 16, 32 or 64 columns: both operands staged through LDS
// step by step, the weights still read exactly once.  Then the same block epilogue as the other producer.
template <typename SH, typename EL>
__global__ __launch_bounds__(64 * kTileWaves) void lmhead_tile_kernel(LmHeadParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  static_assert(SH::ROWS == kRowsPerBlock, "the epilogue's block");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave / SH::WC, wc = wave % SH::WC;
  const int c = lane & 15, g = lane >> 4;
  const int row_base = blockIdx.x * kRowsPerBlock;
  GemmTileArgs t;
  t.w = p.w; t.hidden = p.hidden; t.zeros = p.zeros; t.D = t.pitch = p.D; t.V = p.Vp1; t.row_base = row_base; t.streamed = p.streamed;
  f32x4 acc[SH::RT][SH::CTW];
  tile_product<SH, EL>(t, TileColumns{p.BT}, smem, acc);
  // (the loop's last barrier has every wavefront done with the LDS tiles)
  float* zbuf = (float*)smem;
#pragma unroll
  for (int ct = 0; ct < SH::CTW; ++ct) {
    const int col = (wc * SH::CTW + ct) * 16 + c;
    if (col >= p.BT) continue;
#pragma unroll
    for (int rt = 0; rt < SH::RT; ++rt) {
      f32x4 z;
      const int r0 = (wr * SH::RT + rt) * 16 + g * 4;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = row_base + r0 + i;
        z[i] = row < p.Vp1 ? acc[rt][ct][i] + (p.bias ? p.bias[row] : 0.f) : -INFINITY;
      }
      *(f32x4*)(zbuf + col * kZStride + r0) = z;
    }
  }
  __syncthreads();
  if constexpr (SH::COLS <= 16) {
    // a wavefront per column, at most two in turn (dma_rows: several row blocks)
    if (!SH::DMA && p.n_blocks == 1) lmhead_block_epilogue<true>(p, zbuf);
    else lmhead_block_epilogue<false>(p, zbuf);
  } else {
    unsigned char* part = smem + kMaxCols * kZStride * 4;
    if (p.k <= 1) lmhead_block_epilogue_wide<1>(p, zbuf, part);
    else if (p.k <= 2) lmhead_block_epilogue_wide<2>(p, zbuf, part);
    else if (p.k <= 4) lmhead_block_epilogue_wide<4>(p, zbuf, part);
    else lmhead_block_epilogue_wide<8>(p, zbuf, part);
  }
}
constexpr int kLmEpilogueBytes = kMaxCols * kZStride * 4 + kMfmaWaves / 2 * kMaxCols * (8 + 8 * kMaxTopk);
static_assert(kMaxCols <= 64 && kLmEpilogueBytes <= Tile128x64::LDS_BYTES && kLmEpilogueBytes <= Tile128x32::LDS_BYTES &&
                  16 * kZStride * 4 <= Tile128x16::LDS_BYTES && kLmEpilogueBytes <= Dma128x64::LDS_BYTES &&
                  kLmEpilogueBytes <= Dma128x32::LDS_BYTES && 16 * kZStride * 4 <= Dma128x16::LDS_BYTES,
              "one tile holds every column and the epilogue's partials");

template <typename SH, typename EL>
static hipError_t launch_tile_shape(const LmHeadParams& p, hipStream_t stream) {
  hipLaunchKernelGGL((lmhead_tile_kernel<SH, EL>), dim3(p.n_blocks), dim3(64 * kTileWaves), SH::LDS_BYTES, stream, p);
  return hipGetLastError();
}
template <typename EL>
static hipError_t launch_tile(const LmHeadParams& p, hipStream_t stream) {
  // the narrowest tile that holds the columns: a wavefront without live columns would contract for nothing, which
  // float operands (a sixteenth of the bf16 matrix rate) cannot afford
  auto launch = [&](auto straight, auto tile) {
    if (dma_rows(p.Vp1, p.D, EL::ELEM)) return launch_tile_shape<decltype(straight), EL>(p, stream);
    return rows16(p.D, EL::ELEM) ? launch_tile_shape<Rows16<decltype(tile)>, EL>(p, stream) : launch_tile_shape<decltype(tile), EL>(p, stream);
  };
  if (p.BT <= 16) return launch(Dma128x16{}, Tile128x16{});
  if (p.BT <= 32) return launch(Dma128x32{}, Tile128x32{});
  return launch(Dma128x64{}, Tile128x64{});
}

static void launch_merge(const LmHeadParams& p, hipStream_t stream) {
  if (p.k <= 1) hipLaunchKernelGGL(lmhead_merge_kernel<1>, dim3(p.BT), dim3(64), 0, stream, p);
  else if (p.k <= 2) hipLaunchKernelGGL(lmhead_merge_kernel<2>, dim3(p.BT), dim3(64), 0, stream, p);
  else if (p.k <= 4) hipLaunchKernelGGL(lmhead_merge_kernel<4>, dim3(p.BT), dim3(64), 0, stream, p);
  else hipLaunchKernelGGL(lmhead_merge_kernel<8>, dim3(p.BT), dim3(64), 0, stream, p);
}

int flush_deferred(ctcspec_ctx* ctx) {
  if (!ctx->lm_pending) return CTCSPEC_OK;
  ctx->lm_pending = 0;
  LmHeadParams p = {};
  p.BT = ctx->lm_owed.BT; p.k = ctx->lm_owed.k; p.n_blocks = ctx->lm_owed.n_blocks;
  p.pmax = ctx->lm_pmax; p.psum = ctx->lm_psum; p.pkey = ctx->lm_pkey; p.pstride = ctx->lm_max_blocks;
  p.topk_id = ctx->lm_owed.topk_id; p.topk_logp = ctx->lm_owed.topk_logp; p.lse = ctx->lm_owed.lse;
  launch_merge(p, ctx->stream);
  CTCSPEC_HIP(ctx, hipGetLastError());
  return CTCSPEC_OK;
}

// ev0/ev1, when given, are attached to the launch itself: they take the kernel's own begin and end timestamps (what a
// kernel trace reports), without the dispatch work that a pair of events recorded around the launch also spans.
template <int NT, int STAGES>
static hipError_t launch_mfma(const LmHeadParams& p, int lds_bytes, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1) {
  auto kern = lmhead_bf16_mfma_kernel<NT, STAGES>;
  if (ev0 && ev1)
    hipExtLaunchKernelGGL(kern, dim3(p.n_blocks), dim3(64 * kMfmaWaves), lds_bytes, stream, ev0, ev1, 0, p);
  else
    hipLaunchKernelGGL(kern, dim3(p.n_blocks), dim3(64 * kMfmaWaves), lds_bytes, stream, p);
  return hipGetLastError();
}

template <int NT, int STAGES>
static hipError_t allow_mfma_lds() {
  return hipFuncSetAttribute((const void*)lmhead_bf16_mfma_kernel<NT, STAGES>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kMfmaLdsLimit);
}

template <typename EL, typename... SH>
static hipError_t allow_tile_lds() {
  hipError_t e = hipSuccess;
  ((e = e == hipSuccess ? hipFuncSetAttribute((const void*)lmhead_tile_kernel<SH, EL>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                              SH::LDS_BYTES)
                        : e),
   ...);
  return e;
}
template <typename EL>
static hipError_t allow_tile_lds_all() {
  return allow_tile_lds<EL, Tile128x16, Tile128x32, Tile128x64, Rows16<Tile128x16>, Rows16<Tile128x32>, Rows16<Tile128x64>, Dma128x16,
                        Dma128x32, Dma128x64>();
}

// dynamic LDS limits of this file's kernels, on the current device
static hipError_t allow_large_lds() {
  hipError_t e = allow_mfma_lds<1, 4>();
  if (e == hipSuccess) e = allow_mfma_lds<2, 4>();
  if (e == hipSuccess) e = allow_mfma_lds<3, 4>();
  if (e == hipSuccess) e = allow_mfma_lds<4, 4>();
  if (e == hipSuccess) e = allow_mfma_lds<1, 2>();
  if (e == hipSuccess) e = allow_mfma_lds<2, 2>();
  if (e == hipSuccess) e = allow_mfma_lds<3, 2>();
  if (e == hipSuccess) e = allow_mfma_lds<4, 2>();
  if (e == hipSuccess) e = allow_tile_lds_all<TileBf16>();
  if (e == hipSuccess) e = allow_tile_lds_all<TileF32>();
  if (e == hipSuccess) e = prepare_head_ranges();
  return e;
}

// ---- scratch of the entry point that allocates nothing ------------------------------------------------------------
// The same partial results that ctc_draft_topk keeps in its context's workspace, in a device array of the library
// itself: [256 bytes of zeros][pmax][psum][pkey], laid out as in the context for kStaticMaxBlocks row blocks.  A head cut into
// ranges leaves their sums from pmax on: a call uses one or the other, and calls follow each other in stream order.
// Every GPU the library runs on holds its own copy (8.4 MB) at its own address until the process ends.
constexpr int kStaticMaxBlocks = CTCSPEC_NOALLOC_MAX_VOCAB_ROWS / kRowsPerBlock;
constexpr size_t kScratchZeros = 0;
constexpr size_t kScratchPmax = 256, kScratchPart = kScratchPmax;
constexpr size_t kScratchPsum = kScratchPmax + (size_t)kStaticMaxBlocks * kMaxCols * sizeof(float);
constexpr size_t kScratchPkey = kScratchPsum + (size_t)kStaticMaxBlocks * kMaxCols * sizeof(float);
constexpr size_t kScratchPkeyEnd = kScratchPkey + (size_t)kStaticMaxBlocks * kMaxCols * kMaxTopk * sizeof(unsigned long long);
constexpr size_t kScratchPartEnd = kScratchPart + kDraftPartFloats * sizeof(float);
constexpr size_t kScratchBytes = kScratchPkeyEnd > kScratchPartEnd ? kScratchPkeyEnd : kScratchPartEnd;
static_assert(CTCSPEC_NOALLOC_MAX_VOCAB_ROWS % kRowsPerBlock == 0 && kScratchPkey % 256 == 0 && kScratchPart % 256 == 0, "scratch layout");
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// In host code `scratch` is only a handle for the runtime, not a device address: the address on each device comes
// from hipGetSymbolAddress, once per device, and host code uses that pointer everywhere.
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static unsigned char* g_scratch_ptr[kMaxDevices];

static hipError_t scratch_of_current_device(unsigned char** out, bool* first_use) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (first_use) *first_use = false;
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = (unsigned char*)ptr;
    if (first_use) *first_use = true;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t prepare_draft_topk() {
  // set-up of the allocation-free entry point on this device: address of its scratch, zeros block cleared (the
  // array starts out zeroed and no kernel writes that block; clearing it here costs nothing)
  unsigned char* sp = nullptr;
  hipError_t e = scratch_of_current_device(&sp, nullptr);
  if (e == hipSuccess) e = hipMemset(sp + kScratchZeros, 0, 256);
  if (e != hipSuccess) return e;
  return allow_large_lds();
}

}  // namespace ctcspec

using namespace ctcspec;

// Everything ctc_draft_topk does after its argument checks: producer kernel, then the merge kernel.  `err` receives
// error texts (NULL: the thread's context-less error slot); ev0/ev1 non-null: time the producer kernel; *timed is
// set when they were used.
struct LmScratch {
  float* pmax;
  float* psum;
  unsigned long long* pkey;
  int pstride;
  const void* zeros;
  float* part;  // of a head cut along the hidden dimension
};

static int draft_topk_launch(ctcspec_ctx* err, hipStream_t stream, const LmScratch& sc, hipEvent_t ev0, hipEvent_t ev1,
                             int* timed, bool defer, ctcspec_dtype dt, const void* hidden, const void* w, const float* bias, int B,
                             int T, int D, int Vp1, int k, int32_t* topk_id, float* topk_logp, float* lse,
                             float* logits_out) {
  LmHeadParams p;
  p.hidden = hidden; p.w = w; p.bias = bias;
  p.BT = B * T; p.D = D; p.Vp1 = Vp1; p.k = k;
  p.KC = 0; p.hs_bytes = 0; p.hs_magic = 0; p.zeros = sc.zeros;
  p.n_blocks = (Vp1 + kRowsPerBlock - 1) / kRowsPerBlock;
  p.pmax = sc.pmax; p.psum = sc.psum; p.pkey = sc.pkey; p.pstride = sc.pstride;
  p.topk_id = topk_id; p.topk_logp = topk_logp; p.lse = lse; p.logits_out = logits_out;
  const long long row_bytes = (long long)D * (dt == CTCSPEC_BF16 ? 2 : 4);
  p.streamed = streamed_weights(Vp1 * row_bytes, row_bytes);
  const bool timing = ev0 && ev1;
  // defer: leave the partials and record what is owed (err is the context then); the collapse/tree kernel or
  // flush_deferred does the merge
  auto finish = [&]() -> int {
    if (p.n_blocks == 1) return CTCSPEC_OK;  // it has finished itself
    if (defer) {
      err->lm_owed.BT = p.BT; err->lm_owed.k = p.k; err->lm_owed.n_blocks = p.n_blocks;
      err->lm_owed.topk_id = topk_id; err->lm_owed.topk_logp = topk_logp; err->lm_owed.lse = lse;
      err->lm_pending = 1;
      return CTCSPEC_OK;
    }
    launch_merge(p, stream);
    CTCSPEC_HIP(err, hipGetLastError());
    return CTCSPEC_OK;
  };

  const bool f32 = dt == CTCSPEC_F32;
  HeadRangeParams h;
  h.hidden = hidden; h.w = w; h.zeros = sc.zeros; h.part = sc.part; h.cols = p.BT; h.D = D; h.V = Vp1; h.streamed = p.streamed;
  if (plan_draft_head(h, f32, k)) {
    if (timing) CTCSPEC_HIP(err, hipEventRecord(ev0, stream));
    CTCSPEC_HIP(err, launch_head_ranges(h, f32, stream));
    if (timing) {
      CTCSPEC_HIP(err, hipEventRecord(ev1, stream));
      if (timed) *timed = 1;
    }
    CTCSPEC_HIP(err, k <= 1 ? launch_columns<1>(h, p, stream) : k <= 2 ? launch_columns<2>(h, p, stream)
                     : k <= 4 ? launch_columns<4>(h, p, stream) : launch_columns<8>(h, p, stream));
    return CTCSPEC_OK;  // (nothing of it can be left to the collapse kernel)
  }
  if (dt == CTCSPEC_BF16) {
    if (const int stages = draft_stream_stages(p.BT, D, Vp1)) {
      p.KC = D;
      p.hs_bytes = p.BT * (2 * D + 32);
      p.hs_magic = (unsigned int)((0x100000000ull + (unsigned)(D / 8) - 1) / (unsigned)(D / 8));
      int lds = p.hs_bytes + kMfmaWaves * kWStageBytes;
      int nt = (p.BT + 15) / 16;
      hipError_t e;
      if (stages == 4) {
        switch (nt) {
          case 1: e = launch_mfma<1, 4>(p, lds, stream, ev0, ev1); break;
          case 2: e = launch_mfma<2, 4>(p, lds, stream, ev0, ev1); break;
          case 3: e = launch_mfma<3, 4>(p, lds, stream, ev0, ev1); break;
          default: e = launch_mfma<4, 4>(p, lds, stream, ev0, ev1); break;
        }
      } else {
        switch (nt) {
          case 1: e = launch_mfma<1, 2>(p, lds, stream, ev0, ev1); break;
          case 2: e = launch_mfma<2, 2>(p, lds, stream, ev0, ev1); break;
          case 3: e = launch_mfma<3, 2>(p, lds, stream, ev0, ev1); break;
          default: e = launch_mfma<4, 2>(p, lds, stream, ev0, ev1); break;
        }
      }
      CTCSPEC_HIP(err, e);
      if (timing && timed) *timed = 1;
      return finish();
    }
  }
  // every other shape: both operands step through LDS
  if (timing) CTCSPEC_HIP(err, hipEventRecord(ev0, stream));
  CTCSPEC_HIP(err, dt == CTCSPEC_BF16 ? launch_tile<TileBf16>(p, stream) : launch_tile<TileF32>(p, stream));
  if (timing) {
    CTCSPEC_HIP(err, hipEventRecord(ev1, stream));
    if (timed) *timed = 1;
  }
  return finish();
}

// argument checks shared by the two entry points (`name` prefixes the messages)
static int draft_topk_check(ctcspec_ctx* err, const char* name, ctcspec_dtype dt, const void* hidden, const void* w,
                            int B, int T, int D, int Vp1, int k, const int32_t* topk_id, const float* topk_logp) {
  CTCSPEC_REQUIRE(err, hidden && w && topk_id && topk_logp, CTCSPEC_EINVAL, "%s: null pointer", name);
  CTCSPEC_REQUIRE(err, dt == CTCSPEC_F32 || dt == CTCSPEC_BF16, CTCSPEC_EINVAL, "%s: bad dtype", name);
  CTCSPEC_REQUIRE(err, B > 0 && T > 0 && D > 0 && Vp1 > 0 && k > 0, CTCSPEC_EINVAL, "%s: sizes must be positive", name);
  CTCSPEC_REQUIRE(err, aligned16(hidden) && aligned16(w), CTCSPEC_EINVAL, "%s: hidden and w must be 16-byte aligned",
                  name);
  CTCSPEC_REQUIRE(err, (long long)B * T <= kMaxCols, CTCSPEC_EUNSUPPORTED, "%s: B*T=%lld > %d", name, (long long)B * T,
                  kMaxCols);
  CTCSPEC_REQUIRE(err, k <= Vp1, CTCSPEC_EINVAL, "%s: k=%d > vocabulary rows %d", name, k, Vp1);
  return CTCSPEC_OK;
}

extern "C" int ctc_draft_topk(ctcspec_ctx* ctx, ctcspec_dtype dt, const void* hidden, const void* w,
                              const float* bias, int B, int T, int D, int Vp1, int k, int32_t* topk_id,
                              float* topk_logp, float* lse, float* logits_out) {
  if (!ctx) return CTCSPEC_EINVAL;
  if (const int owed = flush_deferred(ctx)) return owed;  // the partials are about to be overwritten
  const int rc = draft_topk_check(ctx, "ctc_draft_topk", dt, hidden, w, B, T, D, Vp1, k, topk_id, topk_logp);
  if (rc != CTCSPEC_OK) return rc;
  CTCSPEC_REQUIRE(ctx, B <= ctx->lim.max_batch && T <= ctx->lim.max_slots && k <= ctx->lim.max_topk &&
                           Vp1 <= ctx->lim.max_vocab_rows,
                  CTCSPEC_EUNSUPPORTED, "ctc_draft_topk: shape exceeds the context's limits");
  const LmScratch sc = {ctx->lm_pmax, ctx->lm_psum, ctx->lm_pkey, ctx->lm_max_blocks, ctx->zeros, ctx->lm_part};
  return draft_topk_launch(ctx, ctx->stream, sc, ctx->lm_profile ? ctx->lm_ev0 : nullptr,
                           ctx->lm_profile ? ctx->lm_ev1 : nullptr, &ctx->lm_profile_valid, ctx->lm_defer != 0, dt, hidden, w,
                           bias, B, T, D, Vp1, k, topk_id, topk_logp, lse, logits_out);
}

extern "C" int ctc_draft_topk_noalloc(void* hip_stream, ctcspec_dtype dt, const void* hidden, const void* w,
                                      const float* bias, int B, int T, int D, int Vp1, int k, int32_t* topk_id,
                                      float* topk_logp, float* lse, float* logits_out) {
  const char* name = "ctc_draft_topk_noalloc";
  const int rc = draft_topk_check(nullptr, name, dt, hidden, w, B, T, D, Vp1, k, topk_id, topk_logp);
  if (rc != CTCSPEC_OK) return rc;
  CTCSPEC_REQUIRE(nullptr, Vp1 <= CTCSPEC_NOALLOC_MAX_VOCAB_ROWS, CTCSPEC_EUNSUPPORTED,
                  "%s: %d vocabulary rows exceed the %d that the library's static scratch holds partial results for "
                  "(use ctc_draft_topk with a context)",
                  name, Vp1, CTCSPEC_NOALLOC_MAX_VOCAB_ROWS);
  CTCSPEC_REQUIRE(nullptr, k <= CTCSPEC_MAX_TOPK && T <= CTCSPEC_MAX_SLOTS, CTCSPEC_EUNSUPPORTED,
                  "%s: k <= %d and T <= %d required", name, CTCSPEC_MAX_TOPK, CTCSPEC_MAX_SLOTS);
  hipStream_t stream = (hipStream_t)hip_stream;
  unsigned char* sp = nullptr;
  bool first_use = false;
  CTCSPEC_HIP(nullptr, scratch_of_current_device(&sp, &first_use));
  if (first_use) {
    // No context was ever created on this device, so the dynamic LDS limits were never raised: do it now (host-side
    // attribute calls, no allocation).  The zeros block needs nothing: the array starts out zeroed and no kernel
    // writes that block.
    CTCSPEC_HIP(nullptr, allow_large_lds());
  }
  const LmScratch sc = {(float*)(sp + kScratchPmax), (float*)(sp + kScratchPsum),
                        (unsigned long long*)(sp + kScratchPkey), kStaticMaxBlocks, sp + kScratchZeros,
                        (float*)(sp + kScratchPart)};
  return draft_topk_launch(nullptr, stream, sc, nullptr, nullptr, nullptr, false, dt, hidden, w, bias, B, T, D, Vp1, k, topk_id,
                           topk_logp, lse, logits_out);
}
