// verify_head_argmax: the base model's LM head over the hidden states of the tree nodes, reduced to the
// greedy token per node.  kv_commit: append the accepted path's keys and values to the cached context.
//
// The head is the same stream over a [V, D] weight matrix as the draft head, but with up to 128 columns
// (one per tree node) instead of 8, and all that is kept of a column is its best (logit, id) key:
//   * verify_head_kernel         - the tile loop of dma_tile.h (gemm_tile.h): 128 vocabulary rows x 16 to 128 columns per
//                                  workgroup (256 x 128 or 256 x 256 with more columns); all column blocks
//                                  in one launch, those of a row block side by side on one XCD (the weights come
//                                  from HBM once)
//   * verify_head_merge_kernel   - best key over the row blocks -> token id, -1 for rows without a node
//   * verify_head_columns_kernel - vocabularies that do not fill the chip (head_ranges.h): the ranges' sums of a column
//                                  -> its token id
#include <type_traits>

#include "dma_tile.h"
#include "head_ranges.h"

namespace ctcspec {

constexpr int kVhCols = kVerifyCols;            // columns (tree nodes) per pass over the weights
constexpr int kVhWaves = kTileWaves;
// dynamic LDS of a tile shape: the staging buffers, or the logit block (column-major, 4 floats of pad per column, at most
// kVhCols columns at a time) when the caller asks for logits - whichever is larger
template <typename SH>
constexpr int vh_lds_bytes() {
  constexpr int block = (SH::COLS < kVhCols ? SH::COLS : kVhCols) * (SH::ROWS + 4) * 4;
  return SH::LDS_BYTES > block ? SH::LDS_BYTES : block;
}
static_assert(kVhCols == 128 && Tile128x128::COLS == kVhCols && Tile256x128::COLS == kVhCols && Dma256x256::COLS == 2 * kVhCols, "tile shape");
static_assert(vh_lds_bytes<Tile256x128>() <= 160 * 1024 && vh_lds_bytes<Dma256x256>() <= 160 * 1024, "fits the compute unit's LDS");

struct VerifyHeadParams {
  const void* hidden;   // [cols_total][D]
  const void* w;        // [V][D]
  int cols_total;       // all columns of the call, covered in one launch, block by block
  int col_blocks;       // of the tile shape's columns
  int D, V;
  int n_blocks;         // row blocks (of the tile shape's rows: 128 or 256)
  unsigned long long* pkey;  // [blocks of kVhCols columns][n_blocks][kVhCols] best key per (column block, row block, column)
  float* logits_out;    // [cols_total][V] or null
  const void* zeros;    // 256 bytes of zeros
  const int32_t* n_nodes;  // [B]
  int max_nodes;
  int32_t* target;      // [cols_total]
  bool streamed;        // streamed_weights (head_plan.h)
};

// the token of a column's best key; rows of the node table without a node get -1
__device__ __forceinline__ void store_target(const VerifyHeadParams& p, int col, unsigned long long best) {
  const int b = col / p.max_nodes, i = col - b * p.max_nodes;
  int n = p.n_nodes[b];
  n = n < 0 ? 0 : (n > p.max_nodes ? p.max_nodes : n);
  p.target[col] = i < n ? (int32_t)rank_key_index(best) : -1;
}

// ---- the shared tile loop, then the best (logit, id) key per column ----------------------------------------------
template <typename SH, typename EL>
__global__ __launch_bounds__(64 * kVhWaves) void verify_head_kernel(VerifyHeadParams p) {
  constexpr int ROWS = SH::ROWS, CTW = SH::CTW, WR = SH::WR, RT = SH::RT;
  constexpr int ZSTRIDE = ROWS + 4;  // floats per column of the logit block
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int NTHREADS = 64 * kVhWaves;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave / SH::WC, wc = wave % SH::WC;
  const int c = lane & 15, g = lane >> 4;
  // Workgroup -> (row block, column block).  Workgroups are dealt to the 8 XCDs round robin, and each XCD has its
  // own L2: the column blocks of one row block get workgroup numbers that differ by multiples of 8 and are
  // neighbours in dispatch order, so they run on the same XCD at about the same time and the weight tile that the
  // first of them pulls from HBM serves the others from that L2 - one pass over the weights in HBM for any number
  // of columns.  (One column block: row block = workgroup number.)
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const bool alone = p.n_blocks == 1;  // a single row block: its column blocks over all XCDs, nothing to merge
  const int cb = alone ? blockIdx.x : slot % p.col_blocks, rb = alone ? 0 : (slot / p.col_blocks) * 8 + xcd;
  if (rb >= p.n_blocks) return;
  const int col0 = cb * SH::COLS;
  const int cols = p.cols_total - col0 < SH::COLS ? p.cols_total - col0 : SH::COLS;
  const int row_base = rb * ROWS;
  GemmTileArgs t;
  t.w = p.w; t.hidden = (const unsigned char*)p.hidden + (size_t)col0 * p.D * EL::ELEM; t.zeros = p.zeros;
  t.D = t.pitch = p.D; t.V = p.V; t.row_base = row_base; t.streamed = p.streamed;
  f32x4 acc[RT][CTW];
  tile_product<SH, EL>(t, TileColumns{cols}, smem, acc);

  // ---- best (logit, id) key per column ---------------------------------------------------------------------
  // (the loop's last barrier has every wavefront done with the LDS tiles)
  if (p.logits_out) {
    // the logit block goes through LDS so that it leaves in rows of the output
    float* zbuf = (float*)smem;
#pragma unroll
    for (int first = 0; first < SH::COLS; first += kVhCols) {
      const int wcol = wc * 16 * CTW - first;  // this wavefront's columns in the part of kVhCols
      if (wcol >= 0 && wcol < kVhCols)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int ct = 0; ct < CTW; ++ct)
            *(f32x4*)(zbuf + (wcol + ct * 16 + c) * ZSTRIDE + (wr * RT + rt) * 16 + g * 4) = acc[rt][ct];
      __syncthreads();
      const int here = cols - first < kVhCols ? cols - first : kVhCols;
      for (int idx = tid; idx < here * ROWS; idx += NTHREADS) {
        const int m = idx / ROWS, r = idx % ROWS;
        if (row_base + r < p.V) p.logits_out[(size_t)(col0 + first + m) * p.V + row_base + r] = zbuf[m * ZSTRIDE + r];
      }
      __syncthreads();
    }
  }
  // a lane holds 4 RT rows of CTW columns: best of those, then over the 4 lane groups (16 RT rows), then over the
  // WR wavefronts that share the columns
  unsigned long long* kbuf = (unsigned long long*)smem;  // [WR][COLS]
#pragma unroll
  for (int ct = 0; ct < CTW; ++ct) {
    unsigned long long best = 0ull;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = row_base + (wr * RT + rt) * 16 + g * 4 + i;
        const unsigned long long key = row < p.V ? rank_key(acc[rt][ct][i], (unsigned)row) : 0ull;
        best = key > best ? key : best;
      }
    unsigned long long o = __shfl_xor(best, 16);
    best = o > best ? o : best;
    o = __shfl_xor(best, 32);
    best = o > best ? o : best;
    if (g == 0) kbuf[wr * SH::COLS + wc * 16 * CTW + ct * 16 + c] = best;
  }
  __syncthreads();
  if (tid < cols) {
    unsigned long long best = kbuf[tid];
#pragma unroll
    for (int r = 1; r < WR; ++r) {
      const unsigned long long o = kbuf[r * SH::COLS + tid];
      best = o > best ? o : best;
    }
    const int col = col0 + tid;
    if (alone) {
      store_target(p, col, best);
      return;
    }
    p.pkey[((size_t)(col / kVhCols) * p.n_blocks + rb) * kVhCols + col % kVhCols] = best;
  }
}

// best key over the row blocks: one wavefront per column; rows of the node table without a node get -1
__global__ __launch_bounds__(64) void verify_head_merge_kernel(VerifyHeadParams p) {
  const int col = blockIdx.x, lane = threadIdx.x;
  const int m = col % kVhCols;
  const unsigned long long* pk = p.pkey + (size_t)(col / kVhCols) * p.n_blocks * kVhCols;
  unsigned long long best = 0ull;
  for (int b0 = 0; b0 < p.n_blocks; b0 += 256) {
    unsigned long long x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int b = b0 + u * 64 + lane;
      x[u] = b < p.n_blocks ? pk[(size_t)b * kVhCols + m] : 0ull;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) best = x[u] > best ? x[u] : best;
  }
  best = wave_max_u64(best);
  if (lane == 0) store_target(p, col, best);
}

// one workgroup per column: the ranges' sums, the logits' row, the best key
template <int NV>
__global__ __launch_bounds__(kHeadColumnThreads) void verify_head_columns_kernel(HeadRangeParams r, VerifyHeadParams p) {
  __shared__ unsigned long long keys[kHeadColumnThreads / 64];
  const int col = blockIdx.x, tid = threadIdx.x;
  const int b = col / p.max_nodes;
  int n = p.n_nodes[b];
  n = n < 0 ? 0 : (n > p.max_nodes ? p.max_nodes : n);
  const bool node = col - b * p.max_nodes < n;
  if (!node && !p.logits_out) {
    if (tid == 0) p.target[col] = -1;
    return;
  }
  f32x4 z[NV];
  load_head_column<NV>(r, col, z);
  if (p.logits_out) store_head_column<NV>(p.logits_out + (size_t)col * p.V, p.V, z);
  unsigned long long best = 0ull;
#pragma unroll
  for (int j = 0; j < NV; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 4 * (j * kHeadColumnThreads + tid) + i;
      const unsigned long long key = row < p.V ? rank_key(z[j][i], (unsigned)row) : 0ull;
      best = key > best ? key : best;
    }
  best = wave_max_u64(best);
  if ((tid & 63) == 0) keys[tid >> 6] = best;
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int w = 1; w < kHeadColumnThreads / 64; ++w) best = keys[w] > best ? keys[w] : best;
    p.target[col] = node ? (int32_t)rank_key_index(best) : -1;
  }
}

// ---- kv_commit ------------------------------------------------------------------------------------------------
struct KvCommitParams {
  const unsigned char* k_tree;
  const unsigned char* v_tree;
  const int32_t* accept_len;
  const int32_t* accept_nodes;
  const int64_t* kv_off;
  const int32_t* ctx_len;
  unsigned char* k_cache;
  unsigned char* v_cache;
  int32_t* ctx_len_out;
  int T, kv_cap, H, max_nodes;
  int row_bytes;  // dh * element size
  int elem_bytes;
};
// one workgroup per (head, sequence); the path has at most T + 1 rows of row_bytes each
__global__ __launch_bounds__(256) void kv_commit_kernel(KvCommitParams p) {
  const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  int len = p.accept_len[b];
  len = len < 0 ? 0 : (len > p.T ? p.T : len);
  int L = p.ctx_len[b];
  L = L < 0 ? 0 : (L > p.kv_cap ? p.kv_cap : L);
  const size_t cache_head = ((size_t)p.kv_off[b] * p.elem_bytes) + (size_t)h * p.kv_cap * p.row_bytes;
  const size_t tree_head = ((size_t)b * p.H + h) * p.max_nodes * (size_t)p.row_bytes;
  // 16-byte copies need every address a multiple of 16: the offsets and the four base pointers
  const bool vec = (p.row_bytes & 15) == 0 && (cache_head & 15) == 0 &&
                   ((((uintptr_t)p.k_cache | (uintptr_t)p.v_cache | (uintptr_t)p.k_tree | (uintptr_t)p.v_tree) & 15) == 0);
  for (int j = 0; j <= len; ++j) {
    const int node = p.accept_nodes[(size_t)b * (p.T + 1) + j];
    const int pos = L + j;
    if (node < 0 || node >= p.max_nodes || pos >= p.kv_cap) continue;
    const size_t src = tree_head + (size_t)node * p.row_bytes, dst = cache_head + (size_t)pos * p.row_bytes;
    if (vec) {
      for (int q = tid; q < p.row_bytes / 16; q += 256) {
        *(u32x4*)(p.k_cache + dst + q * 16) = *(const u32x4*)(p.k_tree + src + q * 16);
        *(u32x4*)(p.v_cache + dst + q * 16) = *(const u32x4*)(p.v_tree + src + q * 16);
      }
    } else {
      for (int q = tid; q < p.row_bytes; q += 256) {
        p.k_cache[dst + q] = p.k_tree[src + q];
        p.v_cache[dst + q] = p.v_tree[src + q];
      }
    }
  }
  if (h == 0 && tid == 0 && p.ctx_len_out) {
    const int grown = L + len + 1;
    p.ctx_len_out[b] = grown > p.kv_cap ? p.kv_cap : grown;
  }
}

// The tile shapes: those of dma_tile.h where dma_rows says so, else those of gemm_tile.h.
template <typename... SH, typename F>
static hipError_t for_shapes(F&& f) {
  hipError_t e = hipSuccess;
  ((e = e == hipSuccess ? f(SH{}) : e), ...);
  return e;
}
template <typename EL>
static hipError_t allow_lds() {
  return for_shapes<Tile128x16, Tile128x32, Tile128x64, Tile128x128, Tile256x128, Rows16<Tile128x16>, Rows16<Tile128x32>,
                    Rows16<Tile128x64>, Rows16<Tile128x128>, Rows16<Tile256x128>, Dma128x16, Dma128x32, Dma128x64, Dma128x128,
                    Dma256x128, Dma256x256>([](auto shape) {
    using SH = decltype(shape);
    return hipFuncSetAttribute((const void*)verify_head_kernel<SH, EL>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               vh_lds_bytes<SH>());
  });
}
hipError_t prepare_verify_head() {
  const hipError_t e = allow_lds<TileBf16>();
  return e == hipSuccess ? allow_lds<TileF32>() : e;
}

template <typename SH, typename EL>
static hipError_t launch_shape(VerifyHeadParams& p, hipStream_t stream) {
  p.n_blocks = (p.V + SH::ROWS - 1) / SH::ROWS;
  p.col_blocks = (p.cols_total + SH::COLS - 1) / SH::COLS;
  const long long grid = p.n_blocks == 1 ? p.col_blocks : (long long)((p.n_blocks + 7) / 8) * 8 * p.col_blocks;  // the caller has checked the range
  hipLaunchKernelGGL((verify_head_kernel<SH, EL>), dim3((unsigned)grid), dim3(64 * kVhWaves), vh_lds_bytes<SH>(), stream, p);
  return hipGetLastError();
}
// One launch for every column block (the kernel's workgroup numbering keeps a row block's column blocks on one XCD).
// Up to 128 columns: 128-row tiles as narrow as the columns allow - a workgroup per compute unit, the stream from HBM
// sets the pace, and no matrix instruction is spent on dead columns.  More: head_wide_columns in head_plan.h.  A single row
// block (dma_rows says no there) is cut into blocks of 16 columns and finishes itself: 100 rows of 64 float, 128 columns 6.1 -> 3.4 us.
template <typename EL>
static hipError_t launch_head(VerifyHeadParams& p, hipStream_t stream) {
  const bool dma = dma_rows(p.V, p.D, EL::ELEM);
  auto launch = [&](auto straight, auto tile) {
    if (dma) return launch_shape<decltype(straight), EL>(p, stream);
    return rows16(p.D, EL::ELEM) ? launch_shape<Rows16<decltype(tile)>, EL>(p, stream) : launch_shape<decltype(tile), EL>(p, stream);
  };
  if (p.V <= kRowsPerBlock || p.cols_total <= 16) return launch(Dma128x16{}, Tile128x16{});  // (a single block: as many workgroups as the columns give)
  if (p.cols_total <= 32) return launch(Dma128x32{}, Tile128x32{});
  if (p.cols_total <= 64) return launch(Dma128x64{}, Tile128x64{});
  if (p.cols_total <= kVhCols) return launch(Dma128x128{}, Tile128x128{});
  if (dma && head_wide_columns(p.V, p.cols_total) == 256) return launch_shape<Dma256x256, EL>(p, stream);
  return launch(Dma256x128{}, Tile256x128{});
}

}  // namespace ctcspec

using namespace ctcspec;

extern "C" int verify_head_argmax(ctcspec_ctx* ctx, ctcspec_dtype dt, const void* node_hidden, const void* w_base,
                                  const int32_t* n_nodes, int B, int max_nodes, int D, int V,
                                  int32_t* target_argmax, float* logits_out) {
  if (!ctx) return CTCSPEC_EINVAL;
  if (const int owed = flush_deferred(ctx)) return owed;
  CTCSPEC_REQUIRE(ctx, node_hidden && w_base && n_nodes && target_argmax, CTCSPEC_EINVAL,
                  "verify_head_argmax: null pointer");
  CTCSPEC_REQUIRE(ctx, dt == CTCSPEC_F32 || dt == CTCSPEC_BF16, CTCSPEC_EINVAL, "verify_head_argmax: bad dtype");
  CTCSPEC_REQUIRE(ctx, B > 0 && max_nodes > 0 && D > 0 && V > 0, CTCSPEC_EINVAL,
                  "verify_head_argmax: sizes must be positive");
  CTCSPEC_REQUIRE(ctx, aligned16(node_hidden) && aligned16(w_base), CTCSPEC_EINVAL,
                  "verify_head_argmax: node_hidden and w_base must be 16-byte aligned");
  CTCSPEC_REQUIRE(ctx, B <= ctx->lim.max_batch && max_nodes <= ctx->lim.max_nodes && V <= ctx->lim.max_vocab_rows,
                  CTCSPEC_EUNSUPPORTED, "verify_head_argmax: shape exceeds the context's limits");
  const long long row_bytes = (long long)D * (dt == CTCSPEC_BF16 ? 2 : 4);
  VerifyHeadParams p;
  p.hidden = node_hidden; p.w = w_base; p.D = D; p.V = V;
  p.zeros = ctx->zeros; p.pkey = ctx->vh_pkey; p.logits_out = logits_out; p.n_nodes = n_nodes; p.max_nodes = max_nodes;
  p.target = target_argmax; p.streamed = streamed_weights((long long)V * row_bytes, row_bytes);
  const long long cols_total = (long long)B * max_nodes;
  CTCSPEC_REQUIRE(ctx, (cols_total + kVhCols - 1) / kVhCols <= ctx->vh_col_blocks, CTCSPEC_EUNSUPPORTED,
                  "verify_head_argmax: %lld columns exceed the context's workspace", cols_total);
  CTCSPEC_REQUIRE(ctx, ((long long)V / kRowsPerBlock + 8) * ((cols_total + kVhCols - 1) / kVhCols) <= 0x7fffffffLL,
                  CTCSPEC_EUNSUPPORTED, "verify_head_argmax: grid too large");
  p.cols_total = (int)cols_total;
  const bool f32 = dt == CTCSPEC_F32;
  HeadRangeParams r;
  r.hidden = node_hidden; r.w = w_base; r.zeros = ctx->zeros; r.part = ctx->vh_part; r.cols = p.cols_total; r.D = D; r.V = V; r.streamed = p.streamed;
  if (plan_base_head(r, f32)) {
    CTCSPEC_HIP(ctx, launch_head_ranges(r, f32, ctx->stream));
    const hipError_t e = launch_for_rows(V, [&](auto nv) {
      hipLaunchKernelGGL(verify_head_columns_kernel<decltype(nv)::value>, dim3((unsigned)cols_total), dim3(kHeadColumnThreads), 0,
                         ctx->stream, r, p);
      return hipGetLastError();
    });
    CTCSPEC_HIP(ctx, e);
    return CTCSPEC_OK;
  }
  CTCSPEC_HIP(ctx, dt == CTCSPEC_BF16 ? launch_head<TileBf16>(p, ctx->stream) : launch_head<TileF32>(p, ctx->stream));
  if (p.n_blocks > 1) {
    hipLaunchKernelGGL(verify_head_merge_kernel, dim3((unsigned)cols_total), dim3(64), 0, ctx->stream, p);
    CTCSPEC_HIP(ctx, hipGetLastError());
  }
  return CTCSPEC_OK;
}

extern "C" int kv_commit(ctcspec_ctx* ctx, ctcspec_dtype dt, const void* k_tree, const void* v_tree,
                         const int32_t* accept_len, const int32_t* accept_nodes, int T, const int64_t* kv_off,
                         const int32_t* ctx_len, int kv_cap, int B, int H, int dh, int max_nodes, void* k_cache,
                         void* v_cache, int32_t* ctx_len_out) {
  if (!ctx) return CTCSPEC_EINVAL;
  if (const int owed = flush_deferred(ctx)) return owed;
  CTCSPEC_REQUIRE(ctx, k_tree && v_tree && accept_len && accept_nodes && kv_off && ctx_len && k_cache && v_cache,
                  CTCSPEC_EINVAL, "kv_commit: null pointer");
  CTCSPEC_REQUIRE(ctx, dt == CTCSPEC_F32 || dt == CTCSPEC_BF16, CTCSPEC_EINVAL, "kv_commit: bad dtype");
  CTCSPEC_REQUIRE(ctx, B > 0 && H > 0 && dh > 0 && max_nodes > 0 && T > 0 && kv_cap >= 0, CTCSPEC_EINVAL,
                  "kv_commit: sizes must be positive");
  CTCSPEC_REQUIRE(ctx, ctx_len_out != ctx_len, CTCSPEC_EINVAL,
                  "kv_commit: ctx_len_out must not be ctx_len (every head's workgroup reads the old length)");
  CTCSPEC_REQUIRE(ctx, B <= 65535 && T <= CTCSPEC_MAX_SLOTS, CTCSPEC_EUNSUPPORTED,
                  "kv_commit: B <= 65535 and T <= %d required", CTCSPEC_MAX_SLOTS);
  KvCommitParams p;
  p.elem_bytes = dt == CTCSPEC_BF16 ? 2 : 4;
  p.k_tree = (const unsigned char*)k_tree; p.v_tree = (const unsigned char*)v_tree;
  p.accept_len = accept_len; p.accept_nodes = accept_nodes; p.kv_off = kv_off; p.ctx_len = ctx_len;
  p.k_cache = (unsigned char*)k_cache; p.v_cache = (unsigned char*)v_cache; p.ctx_len_out = ctx_len_out;
  p.T = T; p.kv_cap = kv_cap; p.H = H; p.max_nodes = max_nodes; p.row_bytes = dh * p.elem_bytes;
  hipLaunchKernelGGL(kv_commit_kernel, dim3(H, B), dim3(256), 0, ctx->stream, p);
  CTCSPEC_HIP(ctx, hipGetLastError());
  return CTCSPEC_OK;
}
