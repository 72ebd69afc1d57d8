// A tile of a [V, D] x [cols, D]^T product whose rows start on 16-byte boundaries: the loop of the heads and of the draft
// layer's passes.  (Rows that start anywhere: gemm_tile.h.)
//
// 8 wavefronts in a WR x WC grid, RT x CTW MFMA tiles of 16 x 16 each, as in gemm_tile.h.  Both operands go from memory
// straight into LDS (buffer loads with the LDS as their target: no staging registers, no LDS writes by the wavefronts), in steps
// of STEPB bytes of a row, into a ring of NA slots for the weights and one of NB for the hidden states.  A row's 16-byte
// chunk q lies at chunk q ^ (row & 7), or q ^ 2 (row & 7) where rows are 256 bytes: a load writes 64 x 16 consecutive bytes, so rows cannot be padded, and in this order the 16
// lanes that the LDS serves together (l .. l+7 with l+16 .. l+23) read fragments from 64 different banks.
//
// A step: k-block by k-block (64 bytes of a row), the fragments of the next block are read under the products of the
// current one.  Behind the last reads of a step stands its one barrier - its slots are free then, and the wait in front of it
// has seen the next step arrive - and the last block's products cover the requests for the step that takes the slots and the
// first reads of the next one.  Requests, reads and products alternate row of tiles by row of tiles: eight requests in a burst
// hold up the products behind them (256 x 256: 112 us in bursts, 103 spread).
//
// What lies behind the rows, the columns or a row's end has an offset that the hardware's bounds check answers with zeros
// without reading, so every wavefront has the same number of requests per step and the waits count them.  The heads' large tiles
// (UNIFORM) make the requests behind the last step as well, of a buffer without records, and take plain loads only: branches among
// 32 products a block cost 4 to 8 % there (512 columns x 32000 rows of 4096), and nontemporal loads spare nothing (122 us
// both ways when the weights come from memory, 107 against 117 when they are cached).
//
// Bound: what a compute unit takes in.  32000 rows of 4096 bf16, us: 64 columns 42.4 (40.7 for the weights' stream alone), 128
// columns 48.0 (44.6 without the products), 512 columns as 256 x 256 tiles 103 (75 without the products, 73 products alone).  Through
// registers, two LDS buffers and a barrier a step: 48, 52 and 137 (256 x 128).
#pragma once

#include "gemm_tile.h"
#include "head_plan.h"

namespace ctcspec {

template <int WR_, int RT_, int CTW_, int STEPB_, int NA_, int NB_, bool UNIFORM_ = false>
struct DmaShape {
  static constexpr bool DMA = true;
  static constexpr int WR = WR_, WC = kTileWaves / WR_, RT = RT_, CTW = CTW_, STEPB = STEPB_, NA = NA_, NB = NB_;
  static constexpr int ROWS = 16 * RT * WR, COLS = 16 * CTW * WC, KK = STEPB / 64;
  static constexpr bool UNIFORM = UNIFORM_;
  static constexpr int CPR = STEPB / 16, RPI = 64 / CPR;  // chunks of a row, rows that one request of a wavefront covers
  static constexpr int AI = ROWS / RPI / kTileWaves;      // requests of a wavefront per step: weights, hidden states
  static constexpr int BI = (COLS / RPI + kTileWaves - 1) / kTileWaves;
  static constexpr int A_BYTES = ROWS * STEPB, B_BYTES = BI * kTileWaves * 1024;
  static constexpr int LDS_BYTES = NA * A_BYTES + NB * B_BYTES;
  static __device__ __forceinline__ int swizzle(int row) { return CPR == 16 ? (row & 7) * 2 : row & 7; }
  static_assert(WR * WC == kTileWaves && ROWS / RPI % kTileWaves == 0 && KK % 2 == 0 && NA >= NB && NB >= 2, "tile shape");
  static_assert(LDS_BYTES <= 160 * 1024, "fits the compute unit's LDS");
};
using Dma128x16 = DmaShape<8, 1, 1, 256, 4, 3>;
using Dma128x32 = DmaShape<4, 2, 1, 256, 4, 3>;
using Dma128x64 = DmaShape<4, 2, 2, 256, 3, 3>;
using Dma128x128 = DmaShape<2, 4, 2, 256, 3, 2>;
using Dma256x128 = DmaShape<4, 4, 4, 128, 3, 3, true>;
using Dma256x256 = DmaShape<2, 8, 4, 128, 3, 2, true>;

// Rows that lie a multiple of 4096 bytes apart, all workgroups at about the same place of their rows: what is in flight then
// falls on a part of the memory channels.  Successive steps are therefore taken 2048 bytes apart, so that the
// prefetched ones are spread.  A stream of 128 rows a workgroup alone, 32000 rows in all, steps of 256 bytes, us in order / 512 /
// 1024 / 2048 / 4096 bytes apart: pitch 4096 27.5 / 26.2 / 24.3 / 21.8 / -, 8192 53.0 / 48.0 / 44.5 / 40.7 / 56.6, 12288
// 79.6 / 72.1 / 64.3 / 59.2 / 84.5, 16384 116 / 102 / 90 / 89 / 117; at 2048, 5120, 6144, 10240 and 14336 all the same within 2 %,
// at 22016 3 % slower 512 apart.  Another place to start from in every workgroup reaches 38 to 41 at 8192, but gives equal
// rows of different blocks different sums.
__host__ __device__ __forceinline__ int step_segment(size_t pitch, int step_bytes) {
  return pitch % 4096 == 0 ? 2048 / step_bytes : 1;
}

// acc as in gemm_tile; every wavefront of the workgroup (8) must call it; it ends with a barrier behind the last use of LDS.
template <typename SH, typename EL, typename COLUMNS>
__device__ __forceinline__ void dma_tile(const GemmTileArgs& t, const COLUMNS& columns, unsigned char* smem,
                                         f32x4 (&acc)[SH::RT][SH::CTW]) {
#if defined(__HIP_DEVICE_COMPILE__)  // (buffer descriptors exist on the device only)
  constexpr int RT = SH::RT, CTW = SH::CTW, STEPB = SH::STEPB, NA = SH::NA, NB = SH::NB, AI = SH::AI, BI = SH::BI, KK = SH::KK;
  constexpr unsigned int kRecords = 0xfffffc00u, kOutside = 0xfffffd00u;  // (a tile's offsets end below both)
  typedef __attribute__((address_space(3))) void* LdsPtr;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave / SH::WC, wc = wave % SH::WC;
  const int c = lane & 15, g = lane >> 4;
  const size_t pitch = (size_t)t.pitch * EL::ELEM;
  const int row_bytes = t.D * EL::ELEM;
  const int steps = (row_bytes + STEPB - 1) / STEPB, tail = row_bytes - (steps - 1) * STEPB;  // bytes of the last step
  const unsigned char* w = (const unsigned char*)t.w + (size_t)t.row_base * pitch;
  const unsigned char* h = (const unsigned char*)t.hidden;

  // request u of this wavefront covers rows RPI (wave * requests + u) ...; bit u of a tail mask: this lane's chunk lies in the
  // last step's part of the row
  unsigned int woff[AI], hoff[BI];
  unsigned int wtail = 0u, htail = 0u;
  const unsigned int pitch32 = (unsigned)pitch;
  const int r0 = lane / SH::CPR, p0 = lane % SH::CPR;
#pragma unroll
  for (int u = 0; u < AI; ++u) {
    const int r = (wave * AI + u) * SH::RPI + r0, q = p0 ^ SH::swizzle(r);
    woff[u] = r < t.V - t.row_base ? r * pitch32 + q * 16 : kOutside;
    wtail |= q * 16 < tail ? 1u << u : 0u;
  }
  // The place of the next request: its step, that step's place in the row (step_segment), its slot.
  const int seg = step_segment(pitch, STEPB);
  struct Cursor { int step = 0, place = 0, lap = 0, slot = 0; };
  Cursor wn, hn;
  // (two steps of 128 bytes side by side: 64 columns x 4096 41.4 us instead of 47.6, the requests alone)
  constexpr int kRun = STEPB < 256 ? 2 : 1;
  auto advance = [&](Cursor& n, int slots) __attribute__((always_inline)) {
    ++n.step;
    n.slot = n.slot + 1 == slots ? 0 : n.slot + 1;
    n.place += kRun == 1 || seg == 1 ? seg : n.step % kRun ? 1 : seg - kRun + 1;
    if (n.place >= steps) n.place = n.lap += kRun;  // (only where seg > 1 does a request follow)
  };
  const unsigned int lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
  auto request = [&](const unsigned char* base, const Cursor& n, unsigned int off, bool here, unsigned int lds, auto nt)
      __attribute__((always_inline)) {
    const bool valid = !SH::UNIFORM || n.step < steps;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(base + (size_t)n.place * STEPB), 0, valid ? kRecords : 0u, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (LdsPtr)(size_t)lds, 16, here || n.place != steps - 1 ? off : kOutside, 0, 0,
                                             decltype(nt)::value ? 2 : 0);
  };
  // requests [from, to) of the step's BI + AI (hidden states, weights), where there is such a step
  auto requests = [&](int from, int to) __attribute__((always_inline)) {
    auto weights = [&](auto nt) __attribute__((always_inline)) {
#pragma unroll
      for (int v = from; v < to; ++v) {
        const int u = v - BI;
        if (u >= 0 && u < AI) request(w, wn, woff[u >= 0 && u < AI ? u : 0], (wtail >> (u & 31)) & 1u, lds0 + wn.slot * SH::A_BYTES + (wave * AI + u) * 1024, nt);
      }
    };
    if (from < BI && (SH::UNIFORM || hn.step < steps))
#pragma unroll
      for (int u = from; u < to; ++u)
        if (u < BI) request(h, hn, hoff[u < BI ? u : 0], (htail >> u) & 1u, lds0 + NA * SH::A_BYTES + hn.slot * SH::B_BYTES + (wave * BI + u) * 1024, std::false_type{});
    if (to > BI && (SH::UNIFORM || wn.step < steps)) {
      if (!SH::UNIFORM && t.streamed) weights(std::true_type{});
      else weights(std::false_type{});
    }
  };
#pragma unroll
  for (int j = -NA; j < 0; ++j) {
    if (j + NB == 0) {  // (behind the first weights' requests)
#pragma unroll
      for (int u = 0; u < BI; ++u) {
        const int r = (wave * BI + u) * SH::RPI + r0, q = p0 ^ SH::swizzle(r), row = r < SH::COLS ? columns.row_or_none(r) : -1;
        hoff[u] = row >= 0 ? row * pitch32 + q * 16 : kOutside;
        htail |= q * 16 < tail ? 1u << u : 0u;
      }
    }
    if (j + NB >= 0) {
      requests(0, BI);
      advance(hn, NB);
    }
    requests(BI, BI + AI);
    advance(wn, NA);
  }
  // The wait where the barrier of step i stands, for the requests of step i + 1, with `left` = steps - 1 - i steps still to
  // come: younger than they are the hidden states of up to NB - 2 steps and the weights of one more where NA > NB.
  auto arrived = [&](int left) __attribute__((always_inline)) {
    auto wait = [&](auto l) __attribute__((always_inline)) {
      constexpr int L = decltype(l)::value, kH = L - 1 < NB - 2 ? L - 1 : NB - 2, kW = NA == NB ? kH : L - (NA - NB) < kH + 1 ? L - (NA - NB) : kH + 1;
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kW > 0 ? kW : 0) * AI + (kH > 0 ? kH : 0) * BI) : "memory");
    };
    if (SH::UNIFORM || left >= NA) wait(std::integral_constant<int, NA>{});
    else if (NA > 3 && left == 3) wait(std::integral_constant<int, 3>{});
    else if (left == 2) wait(std::integral_constant<int, 2>{});
    else wait(std::integral_constant<int, 1>{});
    lds_barrier();
  };

#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CTW; ++ct) acc[rt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int sw = (g ^ SH::swizzle(c)) * 16;
  const int aoff = (wr * RT * 16 + c) * STEPB + sw, boff = NA * SH::A_BYTES + (wc * CTW * 16 + c) * STEPB + sw;
  int aslot = 0, bslot = 0;
  u32x4 a[2][RT], b[2][CTW];
  auto read_fragment = [&](int f, int kk, int j) __attribute__((always_inline)) {  // the columns' first
    if (j < CTW) b[f][j < CTW ? j : 0] = *(const u32x4*)(smem + bslot * SH::B_BYTES + (boff ^ (kk * 64)) + j * 16 * STEPB);
    else if (j < CTW + RT) a[f][j - CTW < RT ? j - CTW : 0] = *(const u32x4*)(smem + aslot * SH::A_BYTES + (aoff ^ (kk * 64)) + (j - CTW) * 16 * STEPB);
  };
  // Rows of tiles that are taken together: with a single tile a row, its products (of float four, one after the other) would stand alone.
  // 13106 rows of 1536 float, 32 columns 36.5 -> 35.6 us, bf16 tiles of 32 columns 1.5 % in the mean.
  constexpr int kRows = CTW == 1 ? RT : 1, kGroups = RT / kRows;
  constexpr int kReads = (CTW + RT + kGroups - 1) / kGroups, kRequests = (AI + BI + kGroups - 1) / kGroups;  // per group of rows of tiles
  // the products of the fragments in slot f, the reads of block kk for the other slot and, at the end of a step, the requests
  auto block = [&](int f, int kk, auto last) __attribute__((always_inline)) {
#pragma unroll
    for (int rt = 0; rt < kGroups; ++rt) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = rt * kReads; j < (rt + 1) * kReads; ++j) read_fragment(f ^ 1, kk, j);
      if constexpr (decltype(last)::value)
        requests(rt * kRequests < BI + AI ? rt * kRequests : BI + AI, (rt + 1) * kRequests < BI + AI ? (rt + 1) * kRequests : BI + AI);
      // (no fence where four products of float follow one another: requests stand between them, 16 columns x 7367 rows of 2048 30.4 -> 30.1 us)
      if constexpr (!(CTW == 1 && EL::ELEM == 4)) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int ct = 0; ct < CTW; ++ct) acc[rt * kRows + r][ct] = EL::mma(a[f][rt * kRows + r], b[f][ct], acc[rt * kRows + r][ct]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  arrived(steps);
#pragma unroll
  for (int j = 0; j < CTW + RT; ++j) read_fragment(0, 0, j);
  for (int i = 0; i < steps; ++i) {
#pragma unroll
    for (int kk = 0; kk + 1 < KK; ++kk) block(kk & 1, kk + 1, std::false_type{});
    arrived(steps - 1 - i);
    aslot = aslot + 1 == NA ? 0 : aslot + 1;
    bslot = bslot + 1 == NB ? 0 : bslot + 1;
    block((KK - 1) & 1, 0, std::true_type{});  // (behind the last step it reads what nobody uses)
    advance(hn, NB);
    advance(wn, NA);
  }
  // (requests behind the last step have to land before the caller uses the LDS)
  if constexpr (SH::UNIFORM) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  lds_barrier();
#endif
}

template <typename SH, typename EL, typename COLUMNS>
__device__ __forceinline__ void tile_product(const GemmTileArgs& t, const COLUMNS& columns, unsigned char* smem,
                                             f32x4 (&acc)[SH::RT][SH::CTW]) {
  if constexpr (SH::DMA) dma_tile<SH, EL>(t, columns, smem, acc);
  else gemm_tile<4, SH, EL>(t, columns, smem, acc);
}

}  // namespace ctcspec
