// A tile of a [V, D] x [cols, D]^T product, bf16 or float operands, fp32 accumulators, whose rows start at any element
// (hidden sizes that are no multiple of 16 bytes): what the heads take there, and for the smallest calls, and the draft layer for
// its shortest ranges but one.  Others: dma_tile.h.
//
// 8 wavefronts in a WR x WC grid (WR * WC = 8): wavefront (wr, wc) owns weight rows [16 RT wr, +16 RT) x columns
// [16 CTW wc, +16 CTW) - RT x CTW MFMA tiles.  Shapes in use (rows x columns, bytes of a row per step): 128 x 16,
// x 32, x 64 and x 128 with steps of 256 bytes, and 256 x 128 with steps of 128 (4 x 2 wavefronts, 64 x 64 per
// wavefront) for products with several column blocks: per flop it reads two thirds of the fragments from LDS and
// fetches half of the hidden-state tiles from L2.
// Per step both operands go through LDS: the W tile (the A operand) and the hidden states of the step
// (the B operand) are fetched by all threads together with 16-byte loads declared with an element's alignment, DIST steps
// ahead, into rotating register stages, and written to
// one of two LDS buffers while the other one is computed from: one barrier per step.  Within a step the fragment
// reads of the next k-block and the tile writes are issued in front of the MFMAs of the current one and run under them.
// What bounds it (measured, one compute unit): b128 fragment reads at 128 B per clock, b128 writes at 79 B per
// clock - at 128 x 128, per step 192 KB read + 64 KB written = 2300 clocks against 1024 clocks of MFMA and 1.35 us
// (3200 clocks) for the 32 KB of W at the HBM rate, so the LDS work fits under the stream only if nothing
// serialises.  All loads are unconditional and counted (indices clamped; a request past the last step reads a
// block of zeros), so the waits name the loads that stay in flight.
// Hidden sizes that are no whole number of steps: what is left of every row goes first, padded with zeros - through the
// prefetch stages in narrow tiles, unpipelined in wide ones.
#pragma once

#include <type_traits>
#include <utility>

#include "common.h"

namespace ctcspec {

constexpr int kTileWaves = 8;

__device__ __forceinline__ int clamp_int(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// ROWS16: rows start at multiples of 16 bytes, 256 of them within 32-bit offsets (rows16 in head_plan.h).  Otherwise they start at any element: the
// same 16-byte loads, declared with the element's alignment, 64-bit offsets, and a row's end that has to be shifted into place.  119 rows of
// 632 float cut into ranges 5.0 us so, 6.1 as rows that start anywhere.  STREAMED: of those, the weights by nontemporal loads.
template <int WR_, int CTW_, int STEPB_, int RT_ = 4, bool ROWS16_ = false, bool STREAMED_ = false>
struct TileShape {
  static constexpr bool DMA = false, ROWS16 = ROWS16_, STREAMED = STREAMED_;
  static constexpr int WR = WR_, WC = kTileWaves / WR_;  // wavefront grid
  static constexpr int CTW = CTW_, RT = RT_;             // 16-column and 16-row MFMA tiles per wavefront
  static constexpr int STEPB = STEPB_;                   // bytes of a row per step
  static constexpr int ROWS = 16 * RT * WR, COLS = 16 * CTW * WC;
  static constexpr int CPR = STEPB / 16;                 // 16-byte chunks per staged row
  // bytes per staged row: the step's elements + 32.  A 16-byte LDS access of a wavefront is served 16 lanes per
  // clock, lanes {l .. l+7} together with {l+16 .. l+23} (what the conflict counter shows: a fragment read - lane =
  // row c, chunk g - is conflict-free when rows c .. c+7 at chunks g and g+1 fall on 16 different groups of 4
  // banks, i.e. when the pitch is 32 mod 64 bytes; at 128 + 16 bytes every read took one extra clock in four)
  static constexpr int PITCH = STEPB + 32;
  static constexpr int RPP = 64 * kTileWaves / CPR;      // rows that one 16-byte piece per thread covers
  static constexpr int WP = ROWS / RPP, HP = (COLS + RPP - 1) / RPP;  // pieces per thread: W tile, hidden-state tile
  static constexpr int KK = STEPB / 64;                  // k-blocks of 64 bytes per step
  static constexpr int HS_BYTES = HP * RPP * PITCH, BUF_BYTES = HS_BYTES + ROWS * PITCH;
  static constexpr int LDS_BYTES = 2 * BUF_BYTES;
  static_assert(WR * WC == kTileWaves && ROWS % RPP == 0 && (ROWS16 || !STREAMED), "tile shape");
};
template <typename SH>
using Rows16 = TileShape<SH::WR, SH::CTW, SH::STEPB, SH::RT, true>;
using Tile128x16 = TileShape<8, 1, 256, 1>;
using Tile128x32 = TileShape<4, 1, 256, 2>;
using Tile128x64 = TileShape<2, 1, 256>;
using Tile128x128 = TileShape<2, 2, 256>;
using Tile256x128 = TileShape<4, 4, 128>;

// One 64-byte k-block of a 16 x 16 tile: the operands' 16-byte fragments hold row (or column) lane & 15, chunk
// lane >> 4.  bf16: 32 k in one instruction.  float: 16 k in four, instruction i contracting elements i of the four
// chunks - both operands are cut the same way, so the order of k inside the block does not matter.
struct TileBf16 {
  static constexpr int ELEM = 2;
  static __device__ __forceinline__ f32x4 mma(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};
struct TileF32 {
  static constexpr int ELEM = 4;
  static __device__ __forceinline__ f32x4 mma(u32x4 a, u32x4 b, f32x4 c) {
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y[i], c, 0, 0, 0);
    return c;
  }
};

struct GemmTileArgs {
  const void* w;       // [V][pitch], from its first contracted element on
  const void* hidden;  // [..][pitch], likewise
  const void* zeros;   // 256 bytes of zeros
  int D, V;            // contracted elements, weight rows
  int pitch;           // elements from row to row, of both operands
  int row_base;        // first weight row of the tile
  bool streamed = false;  // dma_tile.h: the weights by nontemporal loads
};
// which row of the hidden states a column of the tile is: columns past the end repeat the last one (never read back), or have none
struct TileColumns {
  int cols;
  __device__ __forceinline__ int operator()(int r) const { return r < cols ? r : cols - 1; }
  __device__ __forceinline__ int row_or_none(int r) const { return r < cols ? r : -1; }
};

typedef __attribute__((address_space(1))) u32x4 GlobalU32x4;  // a pointer made from an integer is generic otherwise

// acc[rt][ct][i]: row row_base + 16 (RT wr + rt) + 4 (lane >> 4) + i, column 16 CTW wc + 16 ct + (lane & 15),
// wr = wave / WC, wc = wave % WC.
// Every wavefront of the workgroup (8) must call it; it ends with a barrier after the last read of LDS.
template <int DIST, typename SH, typename EL, typename COLUMNS>
__device__ __forceinline__ void gemm_tile(const GemmTileArgs& t, const COLUMNS& columns, unsigned char* smem,
                                          f32x4 (&acc)[SH::RT][SH::CTW]) {
  constexpr int CTW = SH::CTW, RT = SH::RT, STEPB = SH::STEPB, PITCH = SH::PITCH, CPR = SH::CPR, RPP = SH::RPP;
  constexpr int WP = SH::WP, HP = SH::HP, KK = SH::KK;
  constexpr int WPK = (WP + KK - 1) / KK, HPK = (HP + KK - 1) / KK;  // pieces written to LDS per k-block of the step before
  constexpr int HS_BYTES = SH::HS_BYTES, BUF_BYTES = SH::BUF_BYTES;
  constexpr bool ROWS16 = SH::ROWS16;
  using Offset = std::conditional_t<ROWS16, unsigned int, size_t>;
  struct Packed16 { u32x4 v; } __attribute__((packed, aligned(EL::ELEM)));  // 16 bytes at an element's alignment
  typedef __attribute__((address_space(1))) Packed16 GlobalPacked16;
  constexpr int TRIP = DIST;    // steps per loop trip: stage and buffer static
  static_assert(DIST % 2 == 0, "an even number of stages");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave / SH::WC, wc = wave % SH::WC;
  const int c = lane & 15, g = lane >> 4;
  const int row_base = t.row_base;
  const size_t row_bytes = (size_t)t.D * EL::ELEM, pitch = (size_t)t.pitch * EL::ELEM;
  const int total_steps = (int)(row_bytes / STEPB);
  // LDS: buffer b = hidden-state tile (COLS rows) then W tile (ROWS rows)

  // piece u of a thread: tile row prow + RPP u, 16-byte chunk pchunk, as a byte offset from the tile's first row.
  // A wavefront covers whole rows (4 of 256 bytes or 8 of 128), and
  // the lanes are dealt so that the 16 lanes the LDS serves together write 256 bytes that cover every bank once:
  // both halves of one 256-byte row, or two 128-byte rows 4 apart (4 x 160 bytes = 32 banks further on).
  int prow, pchunk;
  if constexpr (CPR == 16) {
    prow = (tid >> 6) * 4 + ((lane >> 3) & 1) + 2 * (lane >> 5);
    pchunk = (lane & 7) + 8 * ((lane >> 4) & 1);
  } else {
    static_assert(CPR == 8, "rows of 128 or 256 bytes");
    const int j = (lane >> 3) & 7;
    prow = (tid >> 6) * 8 + ((j & 1) | ((j & 2) << 1) | ((j & 4) >> 1));
    pchunk = lane & 7;
  }
  const unsigned int lane_off = pchunk * 16;
  const uintptr_t w_addr = (uintptr_t)t.w + (size_t)row_base * pitch, h_addr = (uintptr_t)t.hidden;
  const uintptr_t z_addr = (uintptr_t)t.zeros;
  Offset woff[WP], hoff[HP];
  const int dst0 = prow * PITCH + pchunk * 16;
#pragma unroll
  for (int u = 0; u < WP; ++u) {
    const int r = prow + RPP * u, last = t.V - 1 - row_base;
    woff[u] = (Offset)(r < last ? r : last) * (Offset)pitch;  // the ragged last block re-reads the last row
  }
#pragma unroll
  for (int u = 0; u < HP; ++u) hoff[u] = (Offset)columns(prow + RPP * u) * (Offset)pitch;
  // A request past the last step still issues its loads, so that every wait counts the same loads: it reads
  // a 256-byte block of zeros (in L2, no HBM traffic) and nothing computes from the result.
  u32x4 wreg[DIST][WP], hreg[DIST][HP];
  auto request = [&](int step, auto stage) __attribute__((always_inline)) {
    constexpr int S = decltype(stage)::value;
    // address arithmetic in integers: a select between pointers would become a branch around each load
    const bool valid = step < total_steps;
    const Offset mask = valid ? ~(Offset)0 : (Offset)0;
    const Offset st = ((Offset)step * (Offset)STEPB) & mask;
    const uintptr_t hb = (valid ? h_addr : z_addr) + st, wb = (valid ? w_addr : z_addr) + st;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < HP; ++u) {
      const uintptr_t a = hb + ((hoff[u] & mask) + lane_off);
      if constexpr (ROWS16) hreg[S][u] = *(const GlobalU32x4*)a;
      else hreg[S][u] = ((const GlobalPacked16*)a)->v;
    }
#pragma unroll
    for (int u = 0; u < WP; ++u) {
      const uintptr_t a = wb + ((woff[u] & mask) + lane_off);
      if constexpr (SH::STREAMED) wreg[S][u] = __builtin_nontemporal_load((const GlobalU32x4*)a);
      else if constexpr (ROWS16) wreg[S][u] = *(const GlobalU32x4*)a;
      else wreg[S][u] = ((const GlobalPacked16*)a)->v;
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // The elements of a row behind its last whole step (tail_bytes of them), zeros behind those: a thread's chunk has tail_n
  // of its bytes in the row.  It is loaded so that it ends with them - every load stays inside its row - and shifted down
  // when it is used, so that nothing waits for it in between.  (A row of less than 16 bytes: element by element.)
  const int tail_bytes = (int)(row_bytes - (size_t)total_steps * STEPB);
  const int tail_n = clamp_int(tail_bytes - pchunk * 16, 0, 16);
  auto tail_load = [&](uintptr_t row) __attribute__((always_inline)) -> u32x4 {
    if constexpr (ROWS16)  // whole chunks
      return *(const GlobalU32x4*)(row + row_bytes - tail_bytes + (tail_n ? pchunk * 16 : 0));
    if (row_bytes >= 16) return ((const GlobalPacked16*)(row + (tail_n ? row_bytes - tail_bytes + pchunk * 16 + tail_n - 16 : 0)))->v;
    using E = std::conditional_t<EL::ELEM == 2, unsigned short, unsigned int>;
    constexpr int PER = 4 / EL::ELEM;  // elements per word
    typedef __attribute__((address_space(1))) E GlobalE;
    u32x4 v = {0u, 0u, 0u, 0u};
    for (int e = 0; e < 4 * PER; ++e) {
      const unsigned int x = e * EL::ELEM < tail_n ? *(const GlobalE*)(row + e * EL::ELEM) : 0u;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] |= e / PER == q ? x << (8 * EL::ELEM * (e % PER)) : 0u;
    }
    return v;
  };
  auto tail_use = [&](u32x4 v) __attribute__((always_inline)) -> u32x4 {
    if (!ROWS16 && row_bytes >= 16 && tail_n > 0 && tail_n < 16) {
      unsigned long long lo = ((unsigned long long)v[1] << 32) | v[0], hi = ((unsigned long long)v[3] << 32) | v[2];
      const int bits = 8 * (16 - tail_n);
      lo = bits >= 64 ? hi >> (bits & 63) : (lo >> bits) | (hi << (64 - bits));
      hi = bits >= 64 ? 0ull : hi >> bits;
      v = u32x4{(unsigned)lo, (unsigned)(lo >> 32), (unsigned)hi, (unsigned)(hi >> 32)};
    }
    return tail_n ? v : u32x4{0u, 0u, 0u, 0u};
  };
  auto commit = [&](auto stage, auto buffer) __attribute__((always_inline)) {
    constexpr int S = decltype(stage)::value, BUF = decltype(buffer)::value;
    unsigned char* hs = smem + BUF * BUF_BYTES;
    unsigned char* ws = hs + HS_BYTES;
#pragma unroll
    for (int u = 0; u < HP; ++u) *(u32x4*)(hs + (dst0 + u * RPP * PITCH)) = hreg[S][u];
#pragma unroll
    for (int u = 0; u < WP; ++u) *(u32x4*)(ws + (dst0 + u * RPP * PITCH)) = wreg[S][u];
  };
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CTW; ++ct) acc[rt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int aoff = (wr * 16 * RT + c) * PITCH + g * 16, boff = (wc * 16 * CTW + c) * PITCH + g * 16;
  // compute one step from LDS buffer BUF; with COMMIT, also write stage S of the registers to the other buffer.
  // Per k-block: the next fragments' reads and that k-block's share of the tile writes are issued, then the MFMAs of
  // the current fragments, under which those LDS operations run.
  auto compute = [&](auto buffer, auto with_commit, auto stage) __attribute__((always_inline)) {
    constexpr int BUF = decltype(buffer)::value, S = decltype(stage)::value;
    constexpr bool COMMIT = decltype(with_commit)::value;
    const unsigned char* hs = smem + BUF * BUF_BYTES;
    const unsigned char* ws = hs + HS_BYTES;
    unsigned char* hs_next = smem + (1 - BUF) * BUF_BYTES;
    unsigned char* ws_next = hs_next + HS_BYTES;
    u32x4 a[2][RT], b[2][CTW];
    auto read_fragments = [&](int kk, int slot) __attribute__((always_inline)) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) a[slot][rt] = *(const u32x4*)(ws + (aoff + rt * 16 * PITCH + kk * 64));
#pragma unroll
      for (int ct = 0; ct < CTW; ++ct)
        b[slot][ct] = *(const u32x4*)(hs + (boff + ct * 16 * PITCH + kk * 64));
    };
    __builtin_amdgcn_sched_barrier(0);
    read_fragments(0, 0);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      __builtin_amdgcn_sched_barrier(0);
      if (kk + 1 < KK) read_fragments(kk + 1, (kk + 1) & 1);
      if constexpr (COMMIT) {
#pragma unroll
        for (int j = 0; j < HPK; ++j) {
          const int u = kk * HPK + j;
          if (u < HP) *(u32x4*)(hs_next + (dst0 + u * RPP * PITCH)) = hreg[S][u < HP ? u : 0];
        }
#pragma unroll
        for (int j = 0; j < WPK; ++j) {
          const int u = kk * WPK + j;
          if (u < WP) *(u32x4*)(ws_next + (dst0 + u * RPP * PITCH)) = wreg[S][u < WP ? u : 0];
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CTW; ++ct) acc[rt][ct] = EL::mma(a[kk & 1][rt], b[kk & 1][ct], acc[rt][ct]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // The pipelined loop takes TRIP steps per trip with no exit in between (an exit inside the trip gives the
  // loop head a second, differently ordered set of loads in flight and the waits there fall back to draining
  // everything).  In front of it go what lies behind a row's last whole step and the total_steps % TRIP steps that do not
  // fill a trip - through the same rotating stages, one copy of the code per remainder, so that every path reaches the
  // loop with the same loads in flight.  Wide tiles have no registers for that (it spilled, +3 us a call): there they run
  // before the first prefetch, a load latency each.  Narrow ones did too: 8 columns x 12547 rows of 1499 bf16
  // elements 27.4 -> 24.1 us, 64 x 14949 of 1234 21.8 -> 16.8, 40 x 18230 of 1280 33.2 -> 32.1 (whole calls).  The copies make the
  // kernels two to four times as large (base head, 128 x 16 bf16: 5.0 -> 16.5 KB); a call runs one of them, and with everything
  // else flushed out of the caches in between the first of these takes 41.0 us with its launches against 47.6, the second 43.5 against 51.6.
  constexpr bool kWide = RT * CTW >= 8;
  const int lead = total_steps % TRIP;
  auto load_tail = [&](auto stage) __attribute__((always_inline)) {
    constexpr int S = decltype(stage)::value;
#pragma unroll
    for (int u = 0; u < HP; ++u) hreg[S][u] = tail_load(h_addr + hoff[u]);
#pragma unroll
    for (int u = 0; u < WP; ++u) wreg[S][u] = tail_load(w_addr + woff[u]);
  };
  auto commit_tail = [&](auto stage, auto buffer) __attribute__((always_inline)) {
    constexpr int S = decltype(stage)::value;
#pragma unroll
    for (int u = 0; u < HP; ++u) hreg[S][u] = tail_use(hreg[S][u]);
#pragma unroll
    for (int u = 0; u < WP; ++u) wreg[S][u] = tail_use(wreg[S][u]);
    commit(stage, buffer);
  };
  using I0 = std::integral_constant<int, 0>;
  // enter the loop behind `lead` steps, L of which are still to be taken: step i of them uses register stage (i - L) mod
  // DIST and LDS buffer (i - L) & 1, as the loop counts them
  auto enter = [&](auto left_tag, auto tail_first) __attribute__((always_inline)) {
    constexpr int L = decltype(left_tag)::value;
    constexpr bool TAIL = decltype(tail_first)::value;
#define CTCSPEC_TILE_STAGE(i) std::integral_constant<int, (((i) - L) % DIST + DIST) % DIST>{}
#define CTCSPEC_TILE_BUFFER(i) std::integral_constant<int, (((i) - L) % 2 + 2) % 2>{}
    const int step0 = lead - L;
    if constexpr (TAIL) load_tail(CTCSPEC_TILE_STAGE(DIST - 1));
    [&]<int... U>(std::integer_sequence<int, U...>) __attribute__((always_inline)) {
      (request(step0 + U, CTCSPEC_TILE_STAGE(U)), ...);
    }(std::make_integer_sequence<int, TAIL ? DIST - 1 : DIST>{});
    if constexpr (TAIL) {
      commit_tail(CTCSPEC_TILE_STAGE(DIST - 1), CTCSPEC_TILE_BUFFER(1));
      request(step0 + DIST - 1, CTCSPEC_TILE_STAGE(DIST - 1));
      lds_barrier();
      compute(CTCSPEC_TILE_BUFFER(1), std::false_type{}, I0{});
    }
    commit(CTCSPEC_TILE_STAGE(0), CTCSPEC_TILE_BUFFER(0));
    request(step0 + DIST, CTCSPEC_TILE_STAGE(0));
    lds_barrier();
    [&]<int... U>(std::integer_sequence<int, U...>) __attribute__((always_inline)) {
      ((compute(CTCSPEC_TILE_BUFFER(U), std::true_type{}, CTCSPEC_TILE_STAGE(U + 1)),
        request(step0 + U + 1 + DIST, CTCSPEC_TILE_STAGE(U + 1)), lds_barrier()),
       ...);
    }(std::make_integer_sequence<int, L>{});
#undef CTCSPEC_TILE_STAGE
#undef CTCSPEC_TILE_BUFFER
  };
  if (kWide || total_steps < 2) {  // (nothing to prefetch either)
    bool used = false;  // LDS has been computed from
    if (tail_bytes > 0) {
      load_tail(I0{});
      commit_tail(I0{}, I0{});
      lds_barrier();
      compute(I0{}, std::false_type{}, I0{});
      used = true;
    }
    for (int i = 0; i < lead; ++i) {
      request(i, I0{});
      if (used) lds_barrier();
      commit(I0{}, I0{});
      lds_barrier();
      compute(I0{}, std::false_type{}, I0{});
      used = true;
    }
    if (used) lds_barrier();  // (also in front of the caller's reuse of the LDS, when no trip follows)
    if constexpr (kWide)
      if (lead < total_steps) enter(I0{}, std::false_type{});
  } else if constexpr (!kWide) {
    [&]<int... N>(std::integer_sequence<int, N...>) __attribute__((always_inline)) {
      ((lead == N ? (tail_bytes > 0 ? enter(std::integral_constant<int, N>{}, std::true_type{})
                                    : enter(std::integral_constant<int, N>{}, std::false_type{}))
                  : void()),
       ...);
    }(std::make_integer_sequence<int, TRIP>{});
  }
  for (int t = lead; t < total_steps; t += TRIP) {
    [&]<int... U>(std::integer_sequence<int, U...>) __attribute__((always_inline)) {
      // step t + U: write step t + U + 1 (after the last step: zeros into the idle buffer), refill its stage
      ((compute(std::integral_constant<int, U & 1>{}, std::true_type{}, std::integral_constant<int, (U + 1) % DIST>{}),
        request(t + U + 1 + DIST, std::integral_constant<int, (U + 1) % DIST>{}), lds_barrier()),
       ...);
    }(std::make_integer_sequence<int, TRIP>{});
  }
}

}  // namespace ctcspec
