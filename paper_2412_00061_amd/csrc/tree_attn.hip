// tree_verify_attn: tree-masked verification attention of the base model, one layer.
//
// Kernels:
//   * tree_attn_bf16_kernel    - bf16 operands, head dimension 128: MFMA for Q.K^T and P.V, online
//                                softmax, K/V tiles shared by the wavefronts of a workgroup through LDS,
//                                optional key splits combined by tree_attn_merge_kernel
//   * tree_attn_few_kernel     - the same for at most 16 query rows: the wavefronts split the keys
//   * tree_attn_any_kernel     - float operands, and bf16 with other head dimensions: the same online softmax on
//                                blocks of 64 query rows, the same key splits and merge
#include <type_traits>
#include <utility>

#include "attn_plan.h"
#include "gemm_tile.h"

namespace ctcspec {

struct AttnParams {
  const void* q;
  const void* k_cache;
  const void* v_cache;
  const int64_t* kv_off;
  const int32_t* ctx_len;
  int kv_cap;
  const void* k_tree;
  const void* v_tree;
  const int32_t* n_nodes;
  const unsigned long long* anc_mask;
  int B, H, dh, max_nodes;
  float scale;
  float* out;
  // optional second form of the output, written instead of `out`: rows [B*max_nodes][H*dh], each value as two
  // bf16 numbers (high part in plane 0, low part in plane 1) - what the draft layer's next matrix product takes
  unsigned short* rows;
  long long rows_plane;  // elements per plane
  long long few_line;    // tree_attn_few_kernel: bytes of K and V beyond which they are read with streaming loads
};

// ---- bf16, dh = 128 -------------------------------------------------------------------------------
// Workgroup = NW wavefronts = one block of 16*QT*CW query nodes of one (sequence, head) and one of S
// splits of the keys.  The wavefronts form CW row groups x KP = NW/CW key parts: wavefront w owns query
// rows [16*QT*rg, 16*QT*(rg+1)) of the block, rg = w % CW, and of every KP consecutive tiles of the
// workgroup the one numbered kp = w / CW (with 64-row blocks two wavefronts per SIMD compute, as with
// 128-row blocks; the two key parts of a row group are joined through LDS at the end).  The keys
// (cached context rows first, then the tree nodes) are cut into tiles of 32; split s takes tiles s,
// s+S, ...  A tile (K and V, 16 KB) is fetched ONCE per workgroup by all threads together (one
// 16-byte load of K and of V per thread and tile, PF iterations ahead in registers), put into one of
// two LDS stages of KP tiles.  With S == 1 the workgroup writes the result; otherwise it
// leaves an unnormalised partial (O, max, sum) per row in the context workspace and
// tree_attn_merge_kernel combines the S partials.
//
// LDS tile layout: 32 rows (keys) of 256 bytes in 16-byte slots.
//   K: slot = chunk ^ (row & 15).  16 lanes reading the same chunk of 16 different rows (the MFMA A
//      operand of K.Q^T: lane = key row, 8 consecutive dh) touch 16 different slots.
//   V: slot = chunk ^ ((row & 7) << 1).  V is read back with ds_read_b64_tr_b16: 16 lanes fetch 8 bytes
//      each from 4 rows x 32 bytes and the instruction hands every lane four CONSECUTIVE KEYS of one dh
//      column - the A operand of O^T += V^T.P - without any shuffling in registers.  With this swizzle
//      the 8 rows x 2 chunks a half wavefront reads lie in 32 different 8-byte bank pairs.
//
// Per tile and wavefront:
//   S^T[key, q] = K.Q^T   : A = K rows from LDS, B = Q^T resident in VGPRs; every K fragment is used
//                           for all QT query tiles
//   P = exp2((S^T - m)*c) : in the MFMA C layout a lane holds 8 keys of ONE query column, so the
//                           running max/sum are per lane plus an exchange between the 4 row groups (ds_bpermute)
//   O^T[dh, q] += V^T.P   : P stays in registers as the B operand, as hi + lo bf16 halves so that it
//                           carries 16 mantissa bits; MFMA row r of output block db is dh = 16*db + r
constexpr int kTileBytes = kTileKeys * 256;        // K or V of one tile
constexpr int kStageBytes = 2 * kTileBytes;        // K then V
// dynamic LDS of the kernel: two stages of KP tiles
constexpr int attn_lds_bytes(int kp) { return 2 * kp * kStageBytes; }

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// (Plain fmaxf on purpose.  As an inline-asm v_max3_f32 this read accumulators of the MFMAs issued right before it,
// and the compiler counts no wait states for inline asm: with the scores consumed straight out of the last product
// the maximum was taken over values that had not landed yet.)
__device__ __forceinline__ float max3_f32(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }
// max / sum over the four lanes l, l^16, l^32, l^48 (the lanes that hold the same query column).
// (v_permlane16_swap / v_permlane32_swap would do this inside the vector ALU, and did in an earlier
// version - with results that changed from run to run in the last bits: the value read right after a
// swap was not always the swapped one.  The exchange goes through ds_bpermute instead.)
__device__ __forceinline__ float max_across_row_groups(float x) {
  x = fmaxf(x, __shfl_xor(x, 16, 64));
  return fmaxf(x, __shfl_xor(x, 32, 64));
}
__device__ __forceinline__ float sum_across_row_groups(float x) {
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}

// fp32 value -> bf16 bits, round to nearest even
__device__ __forceinline__ unsigned int rows_bf16_bits(float f) {
  const unsigned int u = __float_as_uint(f);
  return (u & 0x7fffffffu) > 0x7f800000u ? 0x7fc0u : (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
// four consecutive values of an output row in the two-bf16 form (AttnParams::rows), at element `at` of both planes
__device__ __forceinline__ void store_rows4(const AttnParams& p, size_t at, f32x4 o) {
  unsigned int hi[4], lo[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    hi[i] = rows_bf16_bits(o[i]);
    lo[i] = rows_bf16_bits(o[i] - __uint_as_float(hi[i] << 16));
  }
  *(u32x2*)(p.rows + at) = u32x2{hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16)};
  *(u32x2*)(p.rows + p.rows_plane + at) = u32x2{lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16)};
}

// what a kernel leaves: a template parameter, because the code that a short call has to fetch for the two forms that it does not
// write costs 0.2 us of 5
enum class AttnOut { kRows, kTwoBf16Rows, kPartial };

struct AttnSplit {
  int QB;      // query blocks of 16*QT*CW rows
  int S;       // key splits
  float* po;   // [unit][rows][dh] partial O (unnormalised), unit = ((b*H + h)*QB + qb)*S + s
  float* pm;   // [unit][rows] softmax reference, scaled to the log2 domain
  float* pl;   // [unit][rows] running sum
};

// K and V that do not stay in the 256 MB last-level cache from one call to the next are read with loads that leave no copy
// behind.  What counts is what the call reads (the lengths are known on the device only), not the capacity: 8 sequences x 32
// heads x 64 rows, us with plain / streaming loads, the same caches again and again | caches that went out meanwhile:
//   16 MB 12.5 / 17.9 | 18.3 / 19.1     64 MB 20.1 / 32.8 | 34.9 / 33.0       96 MB 24.9 / 36.5 | 40.3 / 37.6
//   144 MB (ragged) 40.9 / 54.9 | 58.2 / 55.9    256 MB 48.9 / 69.5 | 75.9 / 70.0    375 MB 77.7 / 68.3 | 76.8 / 67.7
// Nothing tells a call which of the two it is.  In a model the other layers' weights and caches pass in between, so large
// calls hardly find anything again; small ones may, and have little to gain otherwise: the line lies where the second
// column's gain has reached 7 %, with room for two calls' caches below it.  At most 16 rows gain next to nothing while the
// caches could stay (144 MB 29.0 / 43.5 | 47.0 / 46.7; 375 MB 68.4 / 61.2 | 69.0 / 63.3): there the line is the whole cache,
// less the weights that the draft layer reads from one of its calls to the next (whole layer, 405 MB of weights: 131 MB of
// caches 152 / 158 |, 144 MB | 183 / 180.5; 103 MB of weights, 139 MB of caches 82.5 / 92 |).
constexpr long long kStreamBytes = 96LL << 20, kStreamBytesFew = 256LL << 20;
__device__ __forceinline__ bool reads_more_than(const AttnParams& p, long long bytes) {
  int rows = 0;
  for (int b = threadIdx.x & 63; b < p.B; b += 64) {
    const int L = p.ctx_len[b];
    rows += L < 0 ? 0 : (L > p.kv_cap ? p.kv_cap : L);
  }
  return (long long)wave_sum_i32(rows) * p.H * 512 > bytes;
}

// 16 bytes of K or V; STREAM: read once and gone
template <bool STREAM>
__device__ __forceinline__ u32x4 load_kv(const unsigned char* a) {
  if constexpr (STREAM) return __builtin_nontemporal_load((const u32x4*)a);
  else return *(const u32x4*)a;
}

template <int QT, int NW, int CW, int PF, bool STREAM, AttnOut OUT>
__device__ __forceinline__ void tree_attn_bf16(const AttnParams& p, const AttnSplit& sp) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int ROWS = 16 * QT * CW;
  constexpr int KP = NW / CW;  // key parts: tiles taken per iteration
  static_assert(NW == 8 && NW % CW == 0 && (KP == 1 || (KP == 2 && QT == 1)), "512 threads fetch a tile; the join of two key parts is written for one query tile");
  constexpr int kIterBytes = KP * kStageBytes;  // one LDS stage
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rg = wave % CW, kp = wave / CW;
  const int c = lane & 15, g = lane >> 4;
  int bid = blockIdx.x;
  const int h = bid % p.H;
  bid /= p.H;
  const int split = bid % sp.S;
  bid /= sp.S;
  const int qb = bid % sp.QB;
  const int b = bid / sp.QB;
  int n = p.n_nodes[b];
  n = n < 1 ? 1 : (n > p.max_nodes ? p.max_nodes : n);
  if (qb * ROWS >= n) return;
  int L = p.ctx_len[b];
  L = L < 0 ? 0 : (L > p.kv_cap ? p.kv_cap : L);

  const size_t node_base = ((size_t)b * p.H + h) * p.max_nodes;
  const unsigned char* kc = (const unsigned char*)p.k_cache + ((size_t)p.kv_off[b] + (size_t)h * p.kv_cap * 128) * 2;
  const unsigned char* vc = (const unsigned char*)p.v_cache + ((size_t)p.kv_off[b] + (size_t)h * p.kv_cap * 128) * 2;
  const unsigned char* kt = (const unsigned char*)p.k_tree + node_base * 256;
  const unsigned char* vt = (const unsigned char*)p.v_tree + node_base * 256;

  const int ctxT = (L + kTileKeys - 1) / kTileKeys, treeT = (n + kTileKeys - 1) / kTileKeys;
  const int NTL = ctxT + treeT;
  const int nloc = split < NTL ? (NTL - split + sp.S - 1) / sp.S : 0;  // my tiles: split, split+S, ...
  const int niter = (nloc + KP - 1) / KP;                              // iterations of KP tiles

  // ---- tile loader: thread -> (row, chunk) of K and of V in each of the iteration's KP tiles ----------
  u32x4 ld[PF][2 * KP];
  const int lrow = tid >> 4, lchunk = tid & 15;
  auto issue = [&](int j, auto set_tag) __attribute__((always_inline)) {
    constexpr int SET = decltype(set_tag)::value;
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      // past the last tile the loads are still issued (on the last tile again, an L2 hit): every wait on
      // an earlier tile can then count on exactly PF-1 younger iterations in flight
      const int jl = KP * j + u;
      const int t = split + (jl < nloc ? jl : nloc - 1) * sp.S;
      const bool tree = t >= ctxT;
      const unsigned char* ks = tree ? kt : kc;
      const unsigned char* vs = tree ? vt : vc;
      const int row0 = (tree ? t - ctxT : t) * kTileKeys, limit = tree ? n : L;
      // tile start as a wavefront-uniform address (scalar arithmetic), the thread's place in the tile as a
      // 32-bit offset: two vector instructions per tile instead of 64-bit address arithmetic per thread
      const unsigned char* kt0 = ks + (size_t)row0 * 256;
      const unsigned char* vt0 = vs + (size_t)row0 * 256;
      const int last = limit - 1 - row0;  // >= 0: rows past the end re-read the last valid row (masked later)
      const unsigned int off = (unsigned int)((lrow < last ? lrow : last) * 256 + lchunk * 16);
      ld[SET][u] = load_kv<STREAM>(kt0 + off);
      ld[SET][KP + u] = load_kv<STREAM>(vt0 + off);
    }
  };
  const int coff_k = lrow * 256 + ((lchunk ^ (lrow & 15)) << 4);
  const int coff_v = kTileBytes + lrow * 256 + ((lchunk ^ ((lrow & 7) << 1)) << 4);
  auto commit = [&](auto set_tag, int stage) __attribute__((always_inline)) {
    constexpr int SET = decltype(set_tag)::value;
    unsigned char* base = smem + stage * kIterBytes;
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      *(u32x4*)(base + u * kStageBytes + coff_k) = ld[SET][u];
      *(u32x4*)(base + u * kStageBytes + coff_v) = ld[SET][KP + u];
    }
  };

  // ---- LDS read addresses --------------------------------------------------------------------------
  // K fragment (kb, kk): row kb*16 + c, chunk kk*4 + g; (row & 15) == c
  int koff[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) koff[kk] = c * 256 + (((kk * 4 + g) ^ c) << 4);
  // The read addresses are kept as complete LDS addresses that the compiler cannot take apart again: as
  // "start of the dynamic LDS block + offset" it recomputes all twelve inside the loop instead of keeping them
  // in registers.
  typedef __attribute__((address_space(3))) unsigned char lds_byte;
  const unsigned int lds0 = (unsigned int)(size_t)(lds_byte*)smem;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    koff[kk] += lds0 + kp * kStageBytes;  // this wavefront's tile of the stage
    asm volatile("" : "+v"(koff[kk]));
  }
  // V, transposing read: lane 16g + s fetches 8 bytes of row kb*16 + 4g + (s >> 2), dh 16db + 4(s & 3)..+3;
  // the 16 lanes of a row group then hold dh 16db + s, keys kb*16 + 4g .. + 3
  int toff[8];
  {
    const int s4 = c >> 2;
    const int x7 = ((4 * (g & 1) + s4) << 1) << 4;  // swizzle term of that row, in bytes
    const int rbase = kTileBytes + (4 * g + s4) * 256 + ((c & 2) ? 16 : 0) + ((c & 1) ? 8 : 0);
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      toff[db] = lds0 + kp * kStageBytes + rbase + ((db << 5) ^ x7);
      asm volatile("" : "+v"(toff[db]));
    }
  }

  // ---- this wavefront's query columns: Q fragments (B operand of K.Q^T) and mask words -------------
  const int qbase = qb * ROWS + rg * 16 * QT;
  const bool live_wave = qbase < n;
  bf16x8 qf[QT][4];
  unsigned long long mw0[QT], mw1[QT];
  const int W = (p.max_nodes + 63) >> 6;
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    const int qi = qbase + qt * 16 + c;
    const int qrow = qi < p.max_nodes ? qi : p.max_nodes - 1;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      qf[qt][kk] = __builtin_bit_cast(
          bf16x8, *(const u32x4*)((const unsigned char*)p.q + (node_base + qrow) * 256 + kk * 64 + g * 16));
    mw0[qt] = 0ull;
    mw1[qt] = 0ull;
    if (qi < n) {
      const unsigned long long* mrow = p.anc_mask + ((size_t)b * p.max_nodes + qi) * W;
      mw0[qt] = mrow[0];
      if (W > 1) mw1[qt] = mrow[1];
    }
  }
  const float sl2 = p.scale * 1.4426950408889634f;

  f32x4 o[QT][8];              // lane (c, g): O[q = c][dh = 16db + 4g + i]
  float m_run[QT], l_run[QT];  // m_run: softmax reference in raw (unscaled) score units
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    m_run[qt] = -INFINITY;
    l_run[qt] = 0.f;
#pragma unroll
    for (int db = 0; db < 8; ++db) o[qt][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  auto compute = [&](int jl, auto stage_tag) __attribute__((always_inline)) {
    const int t = split + jl * sp.S;
    const bool tree = t >= ctxT;
    const int row0 = (tree ? t - ctxT : t) * kTileKeys;
    const bool full = !tree && row0 + kTileKeys <= L;  // every key of the tile is visible to every row
    constexpr int sbase = decltype(stage_tag)::value * kIterBytes;  // folds into the instructions' offset fields
    // S^T = K.Q^T for the two blocks of 16 keys, all query tiles
    f32x4 s[QT][2];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      s[qt][0] = f32x4{0.f, 0.f, 0.f, 0.f};
      s[qt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const bf16x8 a = __builtin_bit_cast(
            bf16x8, *(const __attribute__((address_space(3))) u32x4*)(unsigned int)(koff[kk] + (sbase + kb * 4096)));
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
          s[qt][kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[qt][kk], s[qt][kb], 0, 0, 0);
      }
    // V^T fragments of the tile, one per output block of 16 dh
    s16x8 va[8];
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) s16x4*)(unsigned int)(toff[db] + sbase));
      const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) s16x4*)(unsigned int)(toff[db] + (sbase + 4096)));
      va[db] = s16x8{v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
    }
    // online softmax per query tile
    bf16x8 ph[QT], pl[QT];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      float sv[8];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 4; ++i) sv[kb * 4 + i] = s[qt][kb][i];
      if (!full) {
        // this lane's 8 keys are bits 4g..4g+3 and 16+4g..16+4g+3 of the tile's 32-bit visibility word
        const int left = (tree ? n : L) - row0;  // >= 1 keys of the tile exist
        unsigned int vis = left >= 32 ? 0xffffffffu : ((1u << left) - 1u);
        if (tree) {
          const unsigned long long w = row0 < 64 ? mw0[qt] : mw1[qt];
          vis &= (unsigned int)(w >> (row0 & 63));
        }
        vis >>= 4 * g;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int i = 0; i < 4; ++i) sv[kb * 4 + i] = ((vis >> (kb * 16 + i)) & 1u) ? sv[kb * 4 + i] : -INFINITY;
      }
      const float mx8 = max3_f32(max3_f32(sv[0], sv[1], sv[2]), max3_f32(sv[3], sv[4], sv[5]), fmaxf(sv[6], sv[7]));
      // The softmax reference m_run only has to be NEAR the running max: it is moved (and O, l
      // rescaled) when the tile's max exceeds it by more than 2^8 in the exponent domain, so P stays
      // below 256 and the rescaling of the accumulators - by far the most expensive part of the
      // step - happens about once per wavefront instead of once per tile.  A column's maximum is
      // spread over four lanes, but it exceeds the reference only if one of those lanes' own maxima
      // does: a vote over the wavefront decides whether anything moves, and the exchange between the
      // row groups (two LDS round trips in the middle of the tile's dependency chain) is only made then.
      if (__builtin_amdgcn_ballot_w64((mx8 - m_run[qt]) * sl2 > 8.0f) != 0ull) {
        const float mx = max_across_row_groups(mx8);
        if ((mx - m_run[qt]) * sl2 > 8.0f) {
          const float alpha = __builtin_amdgcn_exp2f((m_run[qt] - mx) * sl2);  // 0 on first use
          l_run[qt] *= alpha;
#pragma unroll
          for (int db = 0; db < 8; ++db) o[qt][db] *= alpha;
          m_run[qt] = mx;
        }
      }
      const float ms = (m_run[qt] > -INFINITY ? m_run[qt] : 0.f) * sl2;
      float psum = 0.f;
      u32x4 hi4, lo4;
#pragma unroll
      for (int jp = 0; jp < 4; ++jp) {
        // P = hi + lo: hi is P cut to its upper 16 bits (a bf16 by construction), lo the rounded rest
        const float p0 = __builtin_amdgcn_exp2f(fmaf(sv[2 * jp], sl2, -ms));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(sv[2 * jp + 1], sl2, -ms));
        psum += p0 + p1;
        const unsigned int u0 = __float_as_uint(p0), u1 = __float_as_uint(p1);
        hi4[jp] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
        const float r0 = p0 - __uint_as_float(u0 & 0xffff0000u);
        const float r1 = p1 - __uint_as_float(u1 & 0xffff0000u);
        const bf16x2 lo = bf16x2{(__bf16)r0, (__bf16)r1};
        lo4[jp] = __builtin_bit_cast(unsigned int, lo);
      }
      ph[qt] = __builtin_bit_cast(bf16x8, hi4);
      pl[qt] = __builtin_bit_cast(bf16x8, lo4);
      l_run[qt] += psum;
    }
    // O^T += V^T.P: the hi products of all dh blocks first, then the lo products, so that consecutive
    // MFMAs never wait for each other's accumulator
#pragma unroll
    for (int db = 0; db < 8; ++db)
#pragma unroll
      for (int qt = 0; qt < QT; ++qt)
        o[qt][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, va[db]), ph[qt], o[qt][db], 0, 0, 0);
#pragma unroll
    for (int db = 0; db < 8; ++db)
#pragma unroll
      for (int qt = 0; qt < QT; ++qt)
        o[qt][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, va[db]), pl[qt], o[qt][db], 0, 0, 0);
  };

  // ---- pipeline: loads PF iterations (of KP tiles) ahead in registers, LDS write one iteration ahead ----
  auto for_each_set = [&](auto&& fn) __attribute__((always_inline)) {
    [&]<int... I>(std::integer_sequence<int, I...>) { (fn(std::integral_constant<int, I>{}), ...); }
    (std::make_integer_sequence<int, PF>{});
  };
  if (nloc > 0) {
    for_each_set([&](auto jj_tag) __attribute__((always_inline)) { issue(decltype(jj_tag)::value, jj_tag); });
    commit(std::integral_constant<int, 0>{}, 0);
    lds_barrier();
    // loads, LDS writes and barriers are free of conditions inside an iteration (tile indices clamped), which is
    // what lets the waits be exact; the unrolled body is left after any of its PF steps
    bool more = true;
    for (int j0 = 0; more; j0 += PF) {
      for_each_set([&](auto jj_tag) __attribute__((always_inline)) {
        constexpr int JJ = decltype(jj_tag)::value;
        const int j = j0 + JJ;
        if (!more) return;
        commit(std::integral_constant<int, (JJ + 1) % PF>{}, (JJ + 1) & 1);
        issue(j + PF, jj_tag);
        if (live_wave && KP * j + kp < nloc) compute(KP * j + kp, std::integral_constant<int, (JJ & 1)>{});
        lds_barrier();  // not __syncthreads(): the prefetched tiles must stay in flight
        more = j + 1 < niter;
      });
    }
  }
  // ---- the two key parts of a row group joined: the upper wavefront hands (O, reference, sum) over in LDS ----
  if constexpr (KP == 2) {
    __syncthreads();  // every tile consumed: the stages are free
    f32x4* xo = (f32x4*)smem;                       // [8 dh blocks][CW * 64 lanes]
    float* xm = (float*)(smem + 8 * CW * 64 * 16);  // [CW * 64] reference, then [CW * 64] sum
    static_assert(8 * CW * 64 * 16 + 2 * CW * 64 * 4 <= attn_lds_bytes(KP), "the hand-over fits the stages");
    const int at = rg * 64 + lane;
    if (kp == 1 && live_wave) {
#pragma unroll
      for (int db = 0; db < 8; ++db) xo[db * (CW * 64) + at] = o[0][db];
      xm[at] = m_run[0];
      xm[CW * 64 + at] = l_run[0];
    }
    __syncthreads();
    if (kp == 1) return;
    if (live_wave) {
      const float m1 = xm[at], l1 = xm[CW * 64 + at];
      const float M = fmaxf(m_run[0], m1);
      // a part that saw no visible key has reference -inf and contributes nothing
      const float a0 = m_run[0] > -INFINITY ? __builtin_amdgcn_exp2f((m_run[0] - M) * sl2) : 0.f;
      const float a1 = m1 > -INFINITY ? __builtin_amdgcn_exp2f((m1 - M) * sl2) : 0.f;
#pragma unroll
      for (int db = 0; db < 8; ++db) o[0][db] = o[0][db] * a0 + xo[db * (CW * 64) + at] * a1;
      l_run[0] = l_run[0] * a0 + l1 * a1;
      m_run[0] = M;
    }
  }
  if (!live_wave) return;

  // ---- results ------------------------------------------------------------------------------------
  const size_t unit = (((size_t)b * p.H + h) * sp.QB + qb) * sp.S + split;
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    const float l = sum_across_row_groups(l_run[qt]);
    const int qr = rg * 16 * QT + qt * 16 + c;  // row inside the block
    const int qg = qb * ROWS + qr;
    if (qg >= n) continue;
    if constexpr (OUT != AttnOut::kPartial) {
      const float inv = 1.0f / l;
      float* dst = p.out + (node_base + qg) * 128 + 4 * g;
      const size_t at = ((size_t)b * p.max_nodes + qg) * ((size_t)p.H * 128) + h * 128 + 4 * g;
#pragma unroll
      for (int db = 0; db < 8; ++db) {
        if constexpr (OUT == AttnOut::kTwoBf16Rows) store_rows4(p, at + 16 * db, o[qt][db] * inv);
        else *(f32x4*)(dst + 16 * db) = o[qt][db] * inv;
      }
    } else {
      // nontemporal: the partials are read once, by another kernel; written through, they do not wait in L2 for
      // the write-back at the kernel's end (0.6 us per launch)
      float* dst = sp.po + (unit * ROWS + qr) * 128 + 4 * g;
#pragma unroll
      for (int db = 0; db < 8; ++db) __builtin_nontemporal_store(o[qt][db], (f32x4*)(dst + 16 * db));
      if (g == 0) {
        sp.pm[unit * ROWS + qr] = m_run[qt] * sl2;  // -inf stays -inf (scale > 0)
        sp.pl[unit * ROWS + qr] = l;
      }
    }
  }
}

// LARGE: the capacity leaves room for more than the line
template <int QT, int NW, int CW, int PF, bool LARGE, AttnOut OUT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void tree_attn_bf16_kernel(AttnParams p, AttnSplit sp) {
  if (LARGE && reads_more_than(p, kStreamBytes)) tree_attn_bf16<QT, NW, CW, PF, true, OUT>(p, sp);
  else tree_attn_bf16<QT, NW, CW, PF, false, OUT>(p, sp);
}

// ---- bf16, dh = 128, at most 16 query rows (the draft module's layer, small trees) -----------------------------------
// One row group, so the eight wavefronts of a workgroup split the KEYS: wavefront w takes the tiles w, w + 8, ... of its
// head on its own - its tile in its own 16 KB of LDS, the next one in flight in registers, no barrier - and
// the eight partial results are joined through LDS at the end.  The layouts and the arithmetic of a tile are those of
// tree_attn_bf16_kernel.  Bound: the K/V stream (8 wavefronts x 16 KB in flight per compute unit), and with ragged
// lengths the longest sequence's workgroups.
constexpr int kFewOPitch = 128 * 4 + 16;
constexpr int kFewLds = kFewWaves * kStageBytes + 2 * kFewWaves * kFewRows * 4;
static_assert(kFewRows * kFewOPitch <= kStageBytes, "a wavefront's result fits where its tile was");

template <bool STREAM>
__device__ __forceinline__ void tree_attn_few(const AttnParams& p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int b = (int)blockIdx.x / p.H, h = (int)blockIdx.x - b * p.H;
  int n = p.n_nodes[b];
  n = n < 1 ? 1 : (n > p.max_nodes ? p.max_nodes : n);
  int L = p.ctx_len[b];
  L = L < 0 ? 0 : (L > p.kv_cap ? p.kv_cap : L);
  const size_t node_base = ((size_t)b * p.H + h) * p.max_nodes;
  const unsigned char* kc = (const unsigned char*)p.k_cache + ((size_t)p.kv_off[b] + (size_t)h * p.kv_cap * 128) * 2;
  const unsigned char* vc = (const unsigned char*)p.v_cache + ((size_t)p.kv_off[b] + (size_t)h * p.kv_cap * 128) * 2;
  const unsigned char* kt = (const unsigned char*)p.k_tree + node_base * 256;
  const unsigned char* vt = (const unsigned char*)p.v_tree + node_base * 256;
  const int ctxT = (L + kTileKeys - 1) / kTileKeys;
  const int NTL = ctxT + 1;  // at most 16 nodes: one tree tile
  const int nloc = wave < NTL ? (NTL - wave + kFewWaves - 1) / kFewWaves : 0;

  unsigned char* ks = smem + wave * kStageBytes;  // this wavefront's tile: K, then V
  u32x4 ld[16];
  const int lrow = lane >> 4, lchunk = lane & 15;
  auto issue = [&](int j) __attribute__((always_inline)) {
    const int t = wave + (j < nloc ? j : nloc - 1) * kFewWaves;
    const bool tree = t >= ctxT;
    const int row0 = (tree ? t - ctxT : t) * kTileKeys, last = (tree ? n : L) - 1 - row0;
    const unsigned char* k0 = (tree ? kt : kc) + (size_t)row0 * 256;
    const unsigned char* v0 = (tree ? vt : vc) + (size_t)row0 * 256;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int r = lrow + 4 * u;  // rows past the end re-read the last valid row (masked later)
      const unsigned int off = (unsigned int)((r < last ? r : last) * 256 + lchunk * 16);
      ld[u] = load_kv<STREAM>(k0 + off);
      ld[8 + u] = load_kv<STREAM>(v0 + off);
    }
  };
  auto commit = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int r = lrow + 4 * u;
      *(u32x4*)(ks + r * 256 + ((lchunk ^ (r & 15)) << 4)) = ld[u];
      *(u32x4*)(ks + kTileBytes + r * 256 + ((lchunk ^ ((r & 7) << 1)) << 4)) = ld[8 + u];
    }
  };
  if (nloc > 0) issue(0);

  const int qrow = c < p.max_nodes ? c : p.max_nodes - 1;
  u32x4 qf[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
    qf[kk] = *(const u32x4*)((const unsigned char*)p.q + (node_base + qrow) * 256 + kk * 64 + g * 16);
  unsigned int mw = 0u;
  if (c < n) mw = (unsigned int)p.anc_mask[(size_t)b * p.max_nodes + c];  // one word per row
  const float sl2 = p.scale * 1.4426950408889634f;

  f32x4 o[8];
#pragma unroll
  for (int db = 0; db < 8; ++db) o[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;

  typedef __attribute__((address_space(3))) unsigned char lds_byte;
  const unsigned int tbase = (unsigned int)(size_t)(lds_byte*)ks + kTileBytes + (4 * g + (c >> 2)) * 256 + ((c & 2) ? 16 : 0) + ((c & 1) ? 8 : 0);
  const unsigned int x7 = ((4 * (g & 1) + (c >> 2)) << 1) << 4;  // swizzle term of that row, in bytes
  for (int j = 0; j < nloc; ++j) {
    commit();
    issue(j + 1);  // (past the last tile: that one again, never used)
    const int t = wave + j * kFewWaves;
    const bool tree = t >= ctxT;
    const int row0 = (tree ? t - ctxT : t) * kTileKeys;
    f32x4 s[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
        s[kb] = TileBf16::mma(*(const u32x4*)(ks + (kb * 16 + c) * 256 + (((kk * 4 + g) ^ c) << 4)), qf[kk], s[kb]);
    u32x4 va[8];
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      const unsigned int at = tbase + ((db << 5) ^ x7);
      const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)at);
      const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(at + 4096u));
      va[db] = __builtin_bit_cast(u32x4, s16x8{v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]});
    }
    float sv[8];
    const int left = (tree ? n : L) - row0;  // >= 1 keys of the tile exist
    unsigned int vis = left >= 32 ? 0xffffffffu : ((1u << left) - 1u);
    if (tree) vis &= mw;
    vis >>= 4 * g;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 4; ++i) sv[kb * 4 + i] = ((vis >> (kb * 16 + i)) & 1u) ? s[kb][i] : -INFINITY;
    const float mx8 = max3_f32(max3_f32(sv[0], sv[1], sv[2]), max3_f32(sv[3], sv[4], sv[5]), fmaxf(sv[6], sv[7]));
    if (__builtin_amdgcn_ballot_w64((mx8 - m_run) * sl2 > 8.0f) != 0ull) {
      const float mx = max_across_row_groups(mx8);
      if ((mx - m_run) * sl2 > 8.0f) {
        const float alpha = __builtin_amdgcn_exp2f((m_run - mx) * sl2);  // 0 on first use
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < 8; ++db) o[db] *= alpha;
        m_run = mx;
      }
    }
    const float ms = (m_run > -INFINITY ? m_run : 0.f) * sl2;
    u32x4 hi, lo;
#pragma unroll
    for (int jp = 0; jp < 4; ++jp) {
      const float p0 = __builtin_amdgcn_exp2f(fmaf(sv[2 * jp], sl2, -ms));
      const float p1 = __builtin_amdgcn_exp2f(fmaf(sv[2 * jp + 1], sl2, -ms));
      l_run += p0 + p1;
      const unsigned int u0 = __float_as_uint(p0), u1 = __float_as_uint(p1);
      hi[jp] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
      const float r0 = p0 - __uint_as_float(u0 & 0xffff0000u), r1 = p1 - __uint_as_float(u1 & 0xffff0000u);
      lo[jp] = __builtin_bit_cast(unsigned int, bf16x2{(__bf16)r0, (__bf16)r1});
    }
#pragma unroll
    for (int db = 0; db < 8; ++db) o[db] = TileBf16::mma(va[db], hi, o[db]);
#pragma unroll
    for (int db = 0; db < 8; ++db) o[db] = TileBf16::mma(va[db], lo, o[db]);
  }

  // ---- the eight parts joined: thread -> (row, four consecutive dh), parts in ascending order -----------------------
  float* pm = (float*)(smem + kFewWaves * kStageBytes);  // [wave][row] reference, then [wave][row] sum
  float* pl = pm + kFewWaves * kFewRows;
  const float l = sum_across_row_groups(l_run);
#pragma unroll
  for (int db = 0; db < 8; ++db) *(f32x4*)(ks + c * kFewOPitch + (16 * db + 4 * g) * 4) = o[db];
  if (g == 0) {
    pm[wave * kFewRows + c] = m_run;
    pl[wave * kFewRows + c] = l;
  }
  __syncthreads();
  const int row = tid >> 5, d4 = (tid & 31) * 4;
  if (row >= n) return;
  float M = -INFINITY, Lt = 0.f;
#pragma unroll
  for (int w = 0; w < kFewWaves; ++w) M = fmaxf(M, pm[w * kFewRows + row]);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < kFewWaves; ++w) {
    const float m = pm[w * kFewRows + row];
    const float f = m > -INFINITY ? __builtin_amdgcn_exp2f((m - M) * sl2) : 0.f;  // a part that saw no visible key: nothing
    Lt += f * pl[w * kFewRows + row];
    acc += *(const f32x4*)(smem + w * kStageBytes + row * kFewOPitch + d4 * 4) * f;
  }
  const f32x4 r = acc * (1.0f / Lt);
  if (p.rows) store_rows4(p, ((size_t)b * p.max_nodes + row) * ((size_t)p.H * 128) + (size_t)h * 128 + d4, r);
  else *(f32x4*)(p.out + (node_base + row) * 128 + d4) = r;
}

template <bool LARGE>
__global__ __launch_bounds__(64 * kFewWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void tree_attn_few_kernel(AttnParams p) {
  if (LARGE && reads_more_than(p, p.few_line)) tree_attn_few<true>(p);
  else tree_attn_few<false>(p);
}

// ---- any head dimension, float or bf16 ---------------------------------------------------------------------------
// Workgroup = 4 wavefronts = one block of 64 query rows of one (sequence, head) and one of S splits of the keys;
// a wavefront owns 16 rows.  Tiles of 32 keys (context first, then the tree) go through two LDS stages, fetched by all
// threads PF tiles ahead in registers.  The head dimension is padded to DHP (16 - float only -, 32, 64, 96 or 128) in LDS and registers
// only: the padding of K is zeroed once, that of V feeds output components that are not written.
//   S^T[key, q] = K.Q^T   64-byte k-blocks as in gemm_tile.h (bf16: one product of 32 k, float: four of 4 k)
//   O^T[dh, q] += V^T.P   a lane holds P of keys 16 kb + 4 g + i in the C layout of S^T, which is the B layout as it is:
//       float: product i of key block kb contracts the keys 16 kb + 4 g + i, g = 0..3; V[key][16 db + c] is one LDS word
//              per lane (row pitch = 16 mod 64 bytes: the four rows a wavefront reads lie 16 banks apart)
//       bf16:  the transposing read of the kernel above (row pitch = an odd multiple of 32 bytes: eight rows x 32 bytes
//              cover every bank once); P goes in as three bf16 numbers, which together hold its 24 mantissa bits - this
//              path has always kept P in float
// Values (V) that are infinite or not a number: in the product 0 x inf carries one to rows that do not see its key, and P in
// parts makes an inf a NaN.  A wavefront that finds its sums not finite forms them again from memory, key by key, keys of
// weight 0 left out (the reference and the sum of the weights do not depend on V).
// Bound: float operands by the matrix rate (157 TFLOP/s), bf16 by latency and the K/V stream.  Measured against one
// workgroup per query row with K/V read by every row (what these shapes took before): 2 sequences x 12 heads x 100
// nodes, 300 to 900 keys, float, head dimension 64: 602-638 -> 16.7-18.7 us a call; four sequences x 15 heads x 64
// nodes over 43 keys, bf16, head dimension 64: 67 -> 10 us.
template <typename EL, int DHP>
struct AnyAttn {
  static constexpr int E = EL::ELEM;
  static constexpr int KPITCH = DHP * E + 32;
  static constexpr int VPITCH = E == 4 ? DHP * 4 + 16 : DHP * 2 + 32;
  static constexpr int STAGE = kTileKeys * (KPITCH + VPITCH);
  static constexpr int THREADS = 256, ROWS = 64;
  static constexpr int NP = (kTileKeys * DHP * E / 16 + THREADS - 1) / THREADS;  // 16-byte pieces per thread of K, of V
  // (4 where the registers allow it is slower by 2.4 % in the mean of 70 shapes of 200 to 4000 positions, long histories
  // included: 4 x 24 heads of 64, 16 rows, 3000 positions 20.2 / 19.3 with 2, 8 x 12 of 80, 64 rows, 2000: 24.6 / 23.2)
  static constexpr int PF = 2;
};

template <typename EL, int DHP, AttnOut OUT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void tree_attn_any_kernel(AttnParams p, AttnSplit sp) {
  using C = AnyAttn<EL, DHP>;
  constexpr int E = C::E, NP = C::NP, PF = C::PF, NB = DHP / 16, KB = DHP * E / 64;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  int bid = blockIdx.x;
  const int h = bid % p.H;
  bid /= p.H;
  const int split = bid % sp.S;
  bid /= sp.S;
  const int qb = bid % sp.QB;
  const int b = bid / sp.QB;
  int n = p.n_nodes[b];
  n = n > p.max_nodes ? p.max_nodes : n;
  if (qb * C::ROWS >= n) return;
  int L = p.ctx_len[b];
  L = L < 0 ? 0 : (L > p.kv_cap ? p.kv_cap : L);
  const int dh = p.dh, row_bytes = dh * E, rc = row_bytes / 16;  // 16-byte chunks per row (dh is a multiple of 8)

  const size_t node_base = ((size_t)b * p.H + h) * p.max_nodes;
  const unsigned char* kc = (const unsigned char*)p.k_cache + ((size_t)p.kv_off[b] + (size_t)h * p.kv_cap * dh) * E;
  const unsigned char* vc = (const unsigned char*)p.v_cache + ((size_t)p.kv_off[b] + (size_t)h * p.kv_cap * dh) * E;
  const unsigned char* kt = (const unsigned char*)p.k_tree + node_base * row_bytes;
  const unsigned char* vt = (const unsigned char*)p.v_tree + node_base * row_bytes;

  const int ctxT = (L + kTileKeys - 1) / kTileKeys, treeT = (n + kTileKeys - 1) / kTileKeys;
  const int NTL = ctxT + treeT;
  const int nloc = split < NTL ? (NTL - split + sp.S - 1) / sp.S : 0;  // my tiles: split, split+S, ...

  // ---- tile loader ----------------------------------------------------------------------------------
  struct Packed16 { u32x4 v; } __attribute__((packed, aligned(E)));
  const int pieces = kTileKeys * rc;
  int prow[NP], pch[NP];
  bool own[NP];
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    const int idx = tid + u * C::THREADS;
    own[u] = idx < pieces;
    const int i = own[u] ? idx : pieces - 1;  // a piece past the end repeats the last one and is not written
    prow[u] = i / rc;
    pch[u] = i - prow[u] * rc;
  }
  u32x4 ld[PF][2 * NP];
  auto issue = [&](int j, auto set_tag) __attribute__((always_inline)) {
    constexpr int SET = decltype(set_tag)::value;
    const int t = split + (j < nloc ? j : nloc - 1) * sp.S;  // past the last tile: that one again, never used
    const bool tree = t >= ctxT;
    const int row0 = (tree ? t - ctxT : t) * kTileKeys, last = (tree ? n : L) - 1 - row0;
    const unsigned char* k0 = (tree ? kt : kc) + (size_t)row0 * row_bytes;
    const unsigned char* v0 = (tree ? vt : vc) + (size_t)row0 * row_bytes;
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      // rows past the end re-read the last valid row (masked later)
      const unsigned int off = (unsigned int)((prow[u] < last ? prow[u] : last) * row_bytes + pch[u] * 16);
      ld[SET][u] = ((const Packed16*)(k0 + off))->v;
      ld[SET][NP + u] = ((const Packed16*)(v0 + off))->v;
    }
  };
  auto commit = [&](auto set_tag, int stage) __attribute__((always_inline)) {
    constexpr int SET = decltype(set_tag)::value;
    unsigned char* base = smem + stage * C::STAGE;
#pragma unroll
    for (int u = 0; u < NP; ++u)
      if (own[u]) {
        *(u32x4*)(base + prow[u] * C::KPITCH + pch[u] * 16) = ld[SET][u];
        *(u32x4*)(base + kTileKeys * C::KPITCH + prow[u] * C::VPITCH + pch[u] * 16) = ld[SET][NP + u];
      }
  };

  // ---- query fragments and mask words ------------------------------------------------------------------
  const int qbase = qb * C::ROWS + wave * 16, qi = qbase + c;
  const bool live_wave = qbase < n;
  u32x4 qf[KB];
  {
    const unsigned char* qrow = (const unsigned char*)p.q + (node_base + (qi < n ? qi : n - 1)) * row_bytes;
#pragma unroll
    for (int kk = 0; kk < KB; ++kk) {
      const int ch = kk * 4 + g;
      const u32x4 v = *(const u32x4*)(qrow + (ch < rc ? ch : 0) * 16);
      qf[kk] = ch < rc ? v : u32x4{0u, 0u, 0u, 0u};
    }
  }
  // bf16 up to 64: the mask words behind the first tiles' requests and without a condition - columns past the tree repeat its last row
  // and are not written, and with one word per row the second is never looked at.  In front of them and under a condition, the
  // wavefront waited for them first: 3 x 8 heads of 64, 16 rows, 7 to 47 positions 4.5 -> 4.0 us (4.3 with four tiles
  // requested ahead); the wider forms and float gain nothing by it.
  constexpr bool kMaskBehind = E == 2 && DHP <= 64;
  const int W = (p.max_nodes + 63) >> 6;
  const unsigned long long* mrow = p.anc_mask + ((size_t)b * p.max_nodes + (qi < n ? qi : n - 1)) * W;
  unsigned long long mw0 = 0ull, mw1 = 0ull;
  if constexpr (!kMaskBehind) {
    if (qi < n) {
      mw0 = mrow[0];
      if (W > 1) mw1 = mrow[1];
    }
  }
  const float sl2 = p.scale * 1.4426950408889634f;

  f32x4 o[NB];  // lane (c, g): O[q = c][dh = 16 db + 4 g + i]
#pragma unroll
  for (int db = 0; db < NB; ++db) o[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;  // reference (scaled, base 2) and this lane's part of the sum

  auto compute = [&](int j, int stage) __attribute__((always_inline)) {
    const int t = split + j * sp.S;
    const bool tree = t >= ctxT;
    const int row0 = (tree ? t - ctxT : t) * kTileKeys;
    const unsigned char* ks = smem + stage * C::STAGE;
    const unsigned char* vs = ks + kTileKeys * C::KPITCH;
    f32x4 s[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int kk = 0; kk < KB; ++kk)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
        s[kb] = EL::mma(*(const u32x4*)(ks + (kb * 16 + c) * C::KPITCH + kk * 64 + g * 16), qf[kk], s[kb]);
    // this lane's 8 keys are bits 4g..4g+3 and 16+4g..16+4g+3 of the tile's 32-bit visibility word
    const int left = (tree ? n : L) - row0;  // >= 1 keys of the tile exist
    unsigned int vis = left >= 32 ? 0xffffffffu : ((1u << left) - 1u);
    if (tree) {
      const unsigned long long w = row0 < 64 ? mw0 : mw1;
      vis &= (unsigned int)(w >> (row0 & 63));
    }
    vis >>= 4 * g;
    float sv[8];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 4; ++i) sv[kb * 4 + i] = ((vis >> (kb * 16 + i)) & 1u) ? s[kb][i] * sl2 : -INFINITY;
    const float mx8 = max3_f32(max3_f32(sv[0], sv[1], sv[2]), max3_f32(sv[3], sv[4], sv[5]), fmaxf(sv[6], sv[7]));
    // lazily moved reference, the exchange only after a vote: as in tree_attn_bf16_kernel
    if (__builtin_amdgcn_ballot_w64(mx8 - m_run > 8.0f) != 0ull) {
      const float mx = max_across_row_groups(mx8);
      if (mx - m_run > 8.0f) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - mx);  // 0 on first use
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < NB; ++db) o[db] *= alpha;
        m_run = mx;
      }
    }
    const float ms = m_run > -INFINITY ? m_run : 0.f;
    float pv[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      // the product is formed again, unrounded (a key whose score is not a number counts as hidden)
      const float e = __builtin_amdgcn_exp2f(fmaf(s[q >> 2][q & 3], sl2, -ms));
      pv[q] = sv[q] > -INFINITY ? e : 0.f;
      l_run += pv[q];
    }
    if constexpr (E == 4) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float* vr = (const float*)(vs + (kb * 16 + 4 * g + i) * C::VPITCH) + c;
#pragma unroll
          for (int db = 0; db < NB; ++db)
            o[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[16 * db], pv[kb * 4 + i], o[db], 0, 0, 0);
        }
    } else {
      u32x4 hi, mid, lo;
#pragma unroll
      for (int jp = 0; jp < 4; ++jp) {
        const float p0 = pv[2 * jp], p1 = pv[2 * jp + 1];
        const float r0 = p0 - __uint_as_float(__float_as_uint(p0) & 0xffff0000u);
        const float r1 = p1 - __uint_as_float(__float_as_uint(p1) & 0xffff0000u);
        hi[jp] = __builtin_amdgcn_perm(__float_as_uint(p1), __float_as_uint(p0), 0x07060302u);
        mid[jp] = __builtin_amdgcn_perm(__float_as_uint(r1), __float_as_uint(r0), 0x07060302u);
        const float q0 = r0 - __uint_as_float(__float_as_uint(r0) & 0xffff0000u);
        const float q1 = r1 - __uint_as_float(__float_as_uint(r1) & 0xffff0000u);
        lo[jp] = __builtin_bit_cast(unsigned int, bf16x2{(__bf16)q0, (__bf16)q1});
      }
      typedef __attribute__((address_space(3))) unsigned char lds_byte;
      const unsigned int v0 = (unsigned int)(size_t)(lds_byte*)vs + (4 * g + (c >> 2)) * C::VPITCH + (c & 3) * 8;
      u32x4 va[NB];
#pragma unroll
      for (int db = 0; db < NB; ++db) {
        const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)(unsigned int)(v0 + db * 32));
        const s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)(unsigned int)(v0 + 16 * C::VPITCH + db * 32));
        va[db] = __builtin_bit_cast(u32x4, s16x8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]});
      }
#pragma unroll
      for (int db = 0; db < NB; ++db) o[db] = EL::mma(va[db], hi, o[db]);
#pragma unroll
      for (int db = 0; db < NB; ++db) o[db] = EL::mma(va[db], mid, o[db]);
#pragma unroll
      for (int db = 0; db < NB; ++db) o[db] = EL::mma(va[db], lo, o[db]);
    }
  };

  if (nloc > 0) {
    auto for_each_set = [&](auto&& fn) __attribute__((always_inline)) {
      [&]<int... I>(std::integer_sequence<int, I...>) { (fn(std::integral_constant<int, I>{}), ...); }
      (std::make_integer_sequence<int, PF>{});
    };
    for_each_set([&](auto st) __attribute__((always_inline)) { issue(decltype(st)::value, st); });
    if constexpr (kMaskBehind) {
      mw0 = mrow[0];
      mw1 = mrow[W - 1];
    }
    if (rc * 16 < DHP * E) {  // zeros behind the head dimension in K's rows, both stages
      const int pad = DHP * E / 16 - rc;
      for (int i = tid; i < 2 * kTileKeys * pad; i += C::THREADS) {
        const int r = i / pad, ch = rc + i - r * pad;
        *(u32x4*)(smem + (r / kTileKeys) * C::STAGE + (r % kTileKeys) * C::KPITCH + ch * 16) = u32x4{0u, 0u, 0u, 0u};
      }
    }
    commit(std::integral_constant<int, 0>{}, 0);
    lds_barrier();
    bool more = true;
    for (int j0 = 0; more; j0 += PF) {
      for_each_set([&](auto jj_tag) __attribute__((always_inline)) {
        constexpr int JJ = decltype(jj_tag)::value;
        const int j = j0 + JJ;
        if (!more) return;
        commit(std::integral_constant<int, (JJ + 1) % PF>{}, (JJ + 1) & 1);
        issue(j + PF, jj_tag);
        if (live_wave) compute(j, JJ & 1);
        lds_barrier();
        more = j + 1 < nloc;
      });
    }
  }
  if (!live_wave) return;
  const size_t unit = (((size_t)b * p.H + h) * sp.QB + qb) * sp.S + split;
  const float l = sum_across_row_groups(l_run);
  if (qi >= n) return;
  struct PackedF4 { f32x4 v; } __attribute__((packed, aligned(4)));
  const int qr = wave * 16 + c;
  constexpr bool kSplit = OUT == AttnOut::kPartial;
  const float f = kSplit ? 1.0f : 1.0f / l;
  float* dst = (kSplit ? sp.po + (unit * C::ROWS + qr) * dh : p.out + (node_base + qi) * dh) + 4 * g;
  const size_t row_at = ((size_t)b * p.max_nodes + qi) * ((size_t)p.H * dh) + (size_t)h * dh + 4 * g;
  auto store = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int db = 0; db < NB; ++db)
      if (16 * db + 4 * g < dh) {
        if constexpr (OUT == AttnOut::kPartial) __builtin_nontemporal_store(o[db], (f32x4*)(dst + 16 * db));
        else if constexpr (OUT == AttnOut::kTwoBf16Rows) store_rows4(p, row_at + 16 * db, o[db] * f);
        else ((PackedF4*)(dst + 16 * db))->v = o[db] * f;
      }
  };
  store();
  if (kSplit && g == 0) {
    sp.pm[unit * C::ROWS + qr] = m_run;
    sp.pl[unit * C::ROWS + qr] = l;
  }
  // not finite: once more (behind everything else - in front of the stores it took the other calls 0.3 us)
  f32x4 probe = {0.f, 0.f, 0.f, 0.f};  // 0 x finite
#pragma unroll
  for (int db = 0; db < NB; ++db) probe += (16 * db + 4 * g < dh ? o[db] : f32x4{0.f, 0.f, 0.f, 0.f}) * 0.f;
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(probe[0] + probe[1] + probe[2] + probe[3] == 0.f)) != 0ull, 0)) {
    using T = std::conditional_t<E == 4, float, unsigned short>;
    const T* qrow = (const T*)p.q + (node_base + qi) * dh;
    const float ms = m_run > -INFINITY ? m_run : 0.f;
#pragma unroll
    for (int db = 0; db < NB; ++db) o[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int j = 0; j < nloc; ++j) {
      const int t = split + j * sp.S;
      const bool tree = t >= ctxT;
      const int row0 = (tree ? t - ctxT : t) * kTileKeys, left = (tree ? n : L) - row0;
      const unsigned int vis = tree ? (unsigned int)((row0 < 64 ? mw0 : mw1) >> (row0 & 63)) : 0xffffffffu;
      for (int key = 0; key < kTileKeys && key < left; ++key) {
        const T* kr = (const T*)(tree ? kt : kc) + (size_t)(row0 + key) * dh;
        const T* vr = (const T*)(tree ? vt : vc) + (size_t)(row0 + key) * dh;
        float s = 0.f;
        for (int e = 0; e < dh; ++e) s = fmaf(load_as_float(qrow + e), load_as_float(kr + e), s);
        const float w = ((vis >> key) & 1u) && s * sl2 > -INFINITY ? __builtin_amdgcn_exp2f(fmaf(s, sl2, -ms)) : 0.f;
#pragma unroll
        for (int db = 0; db < NB; ++db)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (16 * db + 4 * g < dh && w != 0.f) o[db][i] = fmaf(w, load_as_float(vr + 16 * db + 4 * g + i), o[db][i]);
      }
    }
    store();
  }
}

// Combine the S key-split partials of every live query row.  Thread -> (row, 4 consecutive dh), 32
// threads per row, 8 rows per workgroup; eight of a thread's partials are requested before any is used,
// so the kernel costs about one memory round trip per eight splits.  (Letting the split that finishes last do the
// merge inside the attention kernel was measured: one workgroup per query block then pulls all S
// partials through a single compute unit, which takes longer than this second launch.)
constexpr int kMergeThreads = 256;
template <bool MANY>  // more than kMergeParts splits
__global__ __launch_bounds__(kMergeThreads) void tree_attn_merge_kernel(AttnParams p, AttnSplit sp, int rows_shift) {
  const int rows_per_block = 1 << rows_shift;  // 64 or 128 query rows per block
  // grid: (blocks of 8 rows, head of a sequence) - the indices come from the block numbers, not from divisions
  const int tid = threadIdx.x;
  const int row = blockIdx.x * (kMergeThreads / 32) + (tid >> 5);
  const long long bh = blockIdx.y;  // b * H + h
  if (row >= p.max_nodes) return;
  const int b = (int)blockIdx.y / p.H;
  int n = p.n_nodes[b];
  n = n < 1 ? 1 : (n > p.max_nodes ? p.max_nodes : n);
  if (row >= n) return;
  const int qb = row >> rows_shift, qr = row & (rows_per_block - 1);
  const size_t unit0 = ((size_t)bh * sp.QB + qb) * sp.S;
  const int d4 = (tid & 31) * 4, dh = p.dh;
  if (d4 >= dh) return;
  float M = -INFINITY, Lt = 0.f;
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 == 0 || (MANY && s0 < sp.S); s0 += kMergeParts) {
    float pmv[kMergeParts], plv[kMergeParts];
    f32x4 pov[kMergeParts];
#pragma unroll
    for (int i = 0; i < kMergeParts; ++i) {
      const bool on = s0 + i < sp.S;
      const size_t r = (unit0 + (on ? s0 + i : s0)) * rows_per_block + qr;
      pmv[i] = on ? sp.pm[r] : -INFINITY;
      plv[i] = sp.pl[r];
      pov[i] = *(const f32x4*)(sp.po + r * dh + d4);
    }
    const float before = M;
#pragma unroll
    for (int i = 0; i < kMergeParts; ++i) M = fmaxf(M, pmv[i]);
    if (MANY) {
      const float f0 = before > -INFINITY ? __builtin_amdgcn_exp2f(before - M) : 0.f;
      Lt *= f0;
      acc *= f0;
    }
#pragma unroll
    for (int i = 0; i < kMergeParts; ++i) {
      const float f = pmv[i] > -INFINITY ? __builtin_amdgcn_exp2f(pmv[i] - M) : 0.f;
      Lt += f * plv[i];
      acc += pov[i] * f;
    }
  }
  auto store = [&]() __attribute__((always_inline)) {
    const f32x4 o = acc * (1.0f / Lt);
    if (p.rows) {
      const int h = (int)(bh - (long long)b * p.H);
      const size_t at = ((size_t)b * p.max_nodes + row) * ((size_t)p.H * dh) + (size_t)h * dh + d4;
      store_rows4(p, at, o);
    } else {
      *(f32x4*)(p.out + ((size_t)bh * p.max_nodes + row) * dh + d4) = o;
    }
  };
  store();
  // A sum that is not finite is formed again without the parts of weight 0, which add nothing whatever they hold.  (As a select in the loop above, the loads wait for pm: +0.6 us.)
  if (__builtin_expect(!(acc[0] * 0.f + acc[1] * 0.f + acc[2] * 0.f + acc[3] * 0.f == 0.f), 0)) {
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < sp.S; ++s) {
      const size_t r = (unit0 + s) * rows_per_block + qr;
      const float m = sp.pm[r], f = m > -INFINITY ? __builtin_amdgcn_exp2f(m - M) : 0.f;
      if (f != 0.f) acc += *(const f32x4*)(sp.po + r * dh + d4) * f;
    }
    store();
  }
}

static hipError_t launch_merge(const AttnParams& p, const AttnSplit& sp, int rows, hipStream_t stream) {
  const unsigned mblocks = (unsigned)((p.max_nodes + kMergeThreads / 32 - 1) / (kMergeThreads / 32));
  auto kern = sp.S > kMergeParts ? tree_attn_merge_kernel<true> : tree_attn_merge_kernel<false>;
  hipLaunchKernelGGL(kern, dim3(mblocks, (unsigned)(p.B * p.H)), dim3(kMergeThreads), 0, stream, p, sp, rows == 64 ? 6 : 7);
  return hipGetLastError();
}
// whether a call can read more than that: all heads, whole capacity
static bool may_read_more_than(const AttnParams& p, long long bytes) { return (long long)p.B * p.H * p.kv_cap * 512 > bytes; }
template <int QT, int NW, int CW, int PF, bool LARGE, AttnOut OUT>
static hipError_t launch_attn_bf16(const AttnParams& p, const AttnSplit& sp, hipStream_t stream) {
  auto kern = tree_attn_bf16_kernel<QT, NW, CW, PF, LARGE, OUT>;
  const long long blocks = (long long)sp.QB * sp.S * p.H * p.B;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64 * NW), attn_lds_bytes(NW / CW), stream, p, sp);
  hipError_t e = hipGetLastError();
  constexpr int kRows = 16 * QT * CW;
  static_assert(kRows == 64 || kRows == 128, "the merge kernel takes the block size as a shift");
  return e != hipSuccess || OUT != AttnOut::kPartial ? e : launch_merge(p, sp, kRows, stream);
}
template <typename EL, int DHP, AttnOut OUT>
static hipError_t launch_attn_any_dh(const AttnParams& p, const AttnSplit& sp, hipStream_t stream) {
  using C = AnyAttn<EL, DHP>;
  const long long blocks = (long long)sp.QB * sp.S * p.H * p.B;
  hipLaunchKernelGGL((tree_attn_any_kernel<EL, DHP, OUT>), dim3((unsigned)blocks), dim3(C::THREADS), 2 * C::STAGE, stream, p, sp);
  hipError_t e = hipGetLastError();
  return e != hipSuccess || OUT != AttnOut::kPartial ? e : launch_merge(p, sp, 64, stream);
}
template <typename EL, AttnOut OUT>
static hipError_t launch_attn_any(const AttnParams& p, const AttnSplit& sp, hipStream_t stream) {
  if constexpr (EL::ELEM == 4)  // half the products of 32 (bf16: a product contracts 32)
    if (p.dh <= 16) return launch_attn_any_dh<EL, 16, OUT>(p, sp, stream);
  if (p.dh <= 32) return launch_attn_any_dh<EL, 32, OUT>(p, sp, stream);
  if (p.dh <= 64) return launch_attn_any_dh<EL, 64, OUT>(p, sp, stream);
  if (p.dh <= 96) return launch_attn_any_dh<EL, 96, OUT>(p, sp, stream);
  return launch_attn_any_dh<EL, 128, OUT>(p, sp, stream);
}

template <typename F>
static hipError_t launch_for(const AttnParams& p, const AttnSplit& sp, F&& launch) {
  if (sp.S > 1) return launch(std::integral_constant<AttnOut, AttnOut::kPartial>{});
  if (p.rows) return launch(std::integral_constant<AttnOut, AttnOut::kTwoBf16Rows>{});
  return launch(std::integral_constant<AttnOut, AttnOut::kRows>{});
}

// kernels with 64 KB of dynamic LDS or more: the 64-row kernel's two stages of two tiles, and float at 128
template <AttnOut OUT>
static hipError_t allow_lds() {
  auto allow = [](const void* kernel, int bytes) {
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  };
  hipError_t e = allow((const void*)tree_attn_bf16_kernel<1, 8, 4, 2, false, OUT>, attn_lds_bytes(2));
  if (e == hipSuccess) e = allow((const void*)tree_attn_bf16_kernel<1, 8, 4, 2, true, OUT>, attn_lds_bytes(2));
  if constexpr (OUT != AttnOut::kTwoBf16Rows)
    if (e == hipSuccess) e = allow((const void*)tree_attn_any_kernel<TileF32, 128, OUT>, 2 * AnyAttn<TileF32, 128>::STAGE);
  return e;
}
// code of this translation unit loaded onto the current device (context creation calls this: a stage call never
// triggers a load, so it can be the first thing a stream capture records)
hipError_t prepare_tree_attn() {
  hipFuncAttributes attr;
  hipError_t e = hipFuncGetAttributes(&attr, (const void*)tree_attn_merge_kernel<false>);
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute((const void*)tree_attn_few_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, kFewLds);
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void*)tree_attn_few_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kFewLds);
  if (e == hipSuccess) e = allow_lds<AttnOut::kRows>();
  if (e == hipSuccess) e = allow_lds<AttnOut::kTwoBf16Rows>();
  if (e == hipSuccess) e = allow_lds<AttnOut::kPartial>();
  return e;
}

}  // namespace ctcspec

using namespace ctcspec;

int ctcspec::tree_verify_attn_rows(ctcspec_ctx* ctx, ctcspec_dtype dt, const void* q, const void* k_cache,
                                   const void* v_cache, const int64_t* kv_off, const int32_t* ctx_len, int kv_cap,
                                   const void* k_tree, const void* v_tree, const int32_t* n_nodes,
                                   const uint64_t* anc_mask, int B, int H, int dh, int max_nodes, float scale,
                                   float* out, unsigned short* rows, long long rows_plane, long long between) {
  if (!ctx) return CTCSPEC_EINVAL;
  if (const int owed = flush_deferred(ctx)) return owed;
  CTCSPEC_REQUIRE(ctx, q && k_cache && v_cache && kv_off && ctx_len && k_tree && v_tree && n_nodes && anc_mask && (out || rows),
                  CTCSPEC_EINVAL, "tree_verify_attn: null pointer");
  CTCSPEC_REQUIRE(ctx, dt == CTCSPEC_F32 || dt == CTCSPEC_BF16, CTCSPEC_EINVAL, "tree_verify_attn: bad dtype");
  CTCSPEC_REQUIRE(ctx, B > 0 && H > 0 && dh > 0 && max_nodes > 0 && kv_cap >= 0, CTCSPEC_EINVAL,
                  "tree_verify_attn: sizes must be positive");
  CTCSPEC_REQUIRE(ctx, aligned16(q) && aligned16(k_cache) && aligned16(v_cache) && aligned16(k_tree) &&
                           aligned16(v_tree),
                  CTCSPEC_EINVAL, "tree_verify_attn: q/k/v pointers must be 16-byte aligned");
  CTCSPEC_REQUIRE(ctx, dh <= CTCSPEC_MAX_HEAD_DIM && dh % 8 == 0 && max_nodes <= CTCSPEC_MAX_NODES,
                  CTCSPEC_EUNSUPPORTED, "tree_verify_attn: dh<=%d, dh%%8==0, max_nodes<=%d required",
                  CTCSPEC_MAX_HEAD_DIM, CTCSPEC_MAX_NODES);
  CTCSPEC_REQUIRE(ctx, B <= ctx->lim.max_batch && H <= ctx->lim.max_heads && dh <= ctx->lim.max_head_dim &&
                           max_nodes <= ctx->lim.max_nodes,
                  CTCSPEC_EUNSUPPORTED, "tree_verify_attn: shape exceeds the context's limits");
  CTCSPEC_REQUIRE(ctx, B <= 65535 && H <= 65535, CTCSPEC_EUNSUPPORTED, "tree_verify_attn: grid too large");

  AttnParams p;
  p.q = q; p.k_cache = k_cache; p.v_cache = v_cache; p.kv_off = kv_off; p.ctx_len = ctx_len; p.kv_cap = kv_cap;
  p.k_tree = k_tree; p.v_tree = v_tree; p.n_nodes = n_nodes; p.anc_mask = (const unsigned long long*)anc_mask;
  p.B = B; p.H = H; p.dh = dh; p.max_nodes = max_nodes; p.scale = scale; p.out = out;
  p.rows = rows; p.rows_plane = rows_plane;
  p.few_line = kStreamBytesFew - between > kStreamBytes ? kStreamBytesFew - between : kStreamBytes;
  if (dt == CTCSPEC_BF16 && dh == 128) {
    CTCSPEC_REQUIRE(ctx, scale > 0.f, CTCSPEC_EINVAL, "tree_verify_attn: scale must be positive");
    const long long bh = (long long)B * H;
    if (attn_keys_by_wavefront(bh, max_nodes, kv_cap)) {
      // Heads that fill the chip without key splits, and at least a tile per wavefront: 8 sequences of 256 to 2048
      // positions x 32 heads x 16 rows 48.9 -> 43 us, 5 x 32 heads x 8 rows over 300 to 1000 positions 20.5 -> 14.0.  With
      // key splits a wavefront has about one tile and the joins are what is left (one sequence of 2048: 15.6 against
      // 13.7 us), so those calls, and shorter contexts, keep the kernel that fetches a tile with all wavefronts.
      CTCSPEC_REQUIRE(ctx, bh <= 65535, CTCSPEC_EUNSUPPORTED, "tree_verify_attn: grid too large");
      if (may_read_more_than(p, p.few_line))
        hipLaunchKernelGGL(tree_attn_few_kernel<true>, dim3((unsigned)bh), dim3(64 * kFewWaves), kFewLds, ctx->stream, p);
      else
        hipLaunchKernelGGL(tree_attn_few_kernel<false>, dim3((unsigned)bh), dim3(64 * kFewWaves), kFewLds, ctx->stream, p);
      CTCSPEC_HIP(ctx, hipGetLastError());
      return CTCSPEC_OK;
    }
    const AttnShape shape = plan_bf16_128(B, H, max_nodes, kv_cap, ctx->attn_units, rows != nullptr);
    // (up to 16 rows, a single row group: the one-tile-per-iteration kernel, whose first tile is in LDS sooner -
    // 9.1 against 9.9 us for the draft layer's 8 rows)
    const bool rows64 = attn_rows64(shape, max_nodes);
    AttnSplit sp;
    sp.QB = shape.QB;
    sp.S = shape.S;
    sp.po = ctx->attn_po; sp.pm = ctx->attn_pm; sp.pl = ctx->attn_pl;
    CTCSPEC_REQUIRE(ctx, bh * sp.QB * sp.S <= 0x7fffffffLL && bh * max_nodes <= 0x7fffffffLL && bh <= 65535,
                    CTCSPEC_EUNSUPPORTED,
                    "tree_verify_attn: grid too large");
    // (two 64-row blocks share K and V through L2)
    const bool large = sp.QB == 1 && may_read_more_than(p, kStreamBytes);
    const hipError_t e = launch_for(p, sp, [&](auto out_tag) {
      constexpr AttnOut OUT = decltype(out_tag)::value;
      return !rows64 ? launch_attn_bf16<1, 8, 8, 2, false, OUT>(p, sp, ctx->stream)
             : large ? launch_attn_bf16<1, 8, 4, 2, true, OUT>(p, sp, ctx->stream)
                     : launch_attn_bf16<1, 8, 4, 2, false, OUT>(p, sp, ctx->stream);
    });
    CTCSPEC_HIP(ctx, e);
    return CTCSPEC_OK;
  }
  AttnSplit sp;
  const AttnShape shape = plan_any(B, H, max_nodes, kv_cap, dh, dt == CTCSPEC_F32, 2LL * ctx->attn_units, rows != nullptr);
  sp.QB = shape.QB;
  sp.S = shape.S;
  const long long blocks = (long long)B * H * sp.QB;
  sp.po = ctx->attn_po; sp.pm = ctx->attn_pm; sp.pl = ctx->attn_pl;
  CTCSPEC_REQUIRE(ctx, blocks * sp.S <= 0x7fffffffLL, CTCSPEC_EUNSUPPORTED, "tree_verify_attn: grid too large");
  CTCSPEC_REQUIRE(ctx, !rows || dt == CTCSPEC_BF16, CTCSPEC_EUNSUPPORTED, "tree_verify_attn: rows are written from bf16 operands");
  const hipError_t e = launch_for(p, sp, [&](auto out_tag) {
    constexpr AttnOut OUT = decltype(out_tag)::value;
    if (dt == CTCSPEC_BF16) return launch_attn_any<TileBf16, OUT>(p, sp, ctx->stream);
    return launch_attn_any<TileF32, OUT == AttnOut::kTwoBf16Rows ? AttnOut::kRows : OUT>(p, sp, ctx->stream);
  });
  CTCSPEC_HIP(ctx, e);
  return CTCSPEC_OK;
}

extern "C" int tree_verify_attn(ctcspec_ctx* ctx, ctcspec_dtype dt, const void* q, const void* k_cache,
                                const void* v_cache, const int64_t* kv_off, const int32_t* ctx_len, int kv_cap,
                                const void* k_tree, const void* v_tree, const int32_t* n_nodes,
                                const uint64_t* anc_mask, int B, int H, int dh, int max_nodes, float scale,
                                float* out) {
  return ctcspec::tree_verify_attn_rows(ctx, dt, q, k_cache, v_cache, kv_off, ctx_len, kv_cap, k_tree, v_tree, n_nodes,
                                        anc_mask, B, H, dh, max_nodes, scale, out, nullptr, 0, 0);
}
