// tree_verify_attn: query blocks and key splits of a call.  Host code without HIP, so that a test can ask it which way a call
// takes.
#pragma once

namespace ctcspec {

constexpr int kMaxKvSplits = 32;
constexpr int kMergeParts = 8;  // partials that the merge kernel requests together
constexpr int kTileKeys = 32;   // keys of a tile
constexpr int kFewWaves = 8, kFewRows = 16;  // tree_attn_few_kernel: wavefronts that split the keys, query rows at most

struct AttnShape { int QB, S; };  // query blocks, key splits

// bf16, head dimension 128: whether the wavefronts of a workgroup split the keys (tree_attn_few_kernel) - heads that fill the
// chip without key splits, and at least a tile per wavefront
inline bool attn_keys_by_wavefront(long long bh, int max_nodes, int kv_cap) {
  return max_nodes <= kFewRows && bh > 128 && (kv_cap + max_nodes + kTileKeys - 1) / kTileKeys > kFewWaves;
}
// else: blocks of 64 rows (two tiles an iteration) or of 128
inline bool attn_rows64(AttnShape s, int max_nodes) { return s.QB == 2 || (max_nodes <= 64 && max_nodes > kFewRows); }

// ---- launch shapes -------------------------------------------------------------------------------------------------
// A call's time by what it is made of, in us; both kernels take the cheapest (query blocks, key splits).
//   workgroups a compute unit takes in turn x (start of one + iterations x time of one) + what splitting costs
// Splitting costs the merge launch and the partial results, which go through memory.  Before, as many splits were taken as
// fill the chip whatever the merge costs, at most 8, and two blocks of 64 rows as soon as the chip was full.  Measured in HIP
// graphs, us a call before / with this choice:
//   bf16, 128: 2 x 40 heads, 128 rows, 128 positions 17.1 (2 splits) / 10.0 (none, two blocks)    6 x 32 heads, 200: 22.3 / 16.8
//     (one block)    4 x 32 heads, 100 rows, 300: 18.5 (2) / 13.2 (1)    32 heads, 64 rows, 256: 11.9 (2) / 10.2 (1)
//     32 heads, 128 rows, 2048 positions: 4 splits both; none 36.8, 2 26.0, 3 21.6, 4 19.6, 8 of one block 20.0
//   bf16, 80: 4 x 16 heads, 50 rows, 93 positions 10.5 (2) / 7.6 (1)    64: 32 heads, 128 rows, 512: 14.6 (8) / 11.9 (4)
//   float, 128: 14 heads, 35 rows, up to 1923 positions 24.4 (8) / 18.4 (18)    float, 16: 4 heads, 128 rows, 32: 7.4 (3) / 4.0 (1, padded
//     to 16 instead of 32)
// Over 400 shapes drawn from 1 to 8 sequences of 4 to 40 heads and 1 to 128 rows over 4 to 2048 positions: 7 % in the mean.
// the merge launch, the partial results' way through memory, and a round trip of the merge for every eight splits more.  Rows as
// two bf16 numbers are the merge's work otherwise: the 2 x 8 rows of a layer of 1024, 300 positions, 42.2 us with the layer's
// attention in two splits, 44.0 in none.
constexpr double kTwoBf16Us = 1.5;
inline double split_us(long long bh, int S, int rows, int dh, bool two_bf16) {
  return S == 1 ? (two_bf16 ? kTwoBf16Us : 0.0) : 3.3 + (double)bh * S * rows * dh * 4 * 0.25e-6 + (S - 1) / kMergeParts * 3.0;
}
// how much longer than one workgroup a compute unit with `load` of them takes.  Of several sequences, not all are the longest.
inline double taking_turns(double load, double next) { return load <= 1.0 ? 1.0 : 1.0 + (load - 1.0) * next; }
// (two at a time hide each other's waits)
inline double side_by_side(double load) { return load <= 1.0 ? 1.0 : load <= 2.0 ? 1.0 + (load - 1.0) * 0.4 : load * 0.7; }
// tiles of 32 keys that a workgroup expects: the lengths are on the device, the host takes most of the capacity for them;
// what does not divide leaves half an iteration idle on average
inline double iterations(int kv_cap, int max_nodes, int S, int per_iter) {
  const double n = (0.875 * kv_cap + max_nodes) / (kTileKeys * per_iter * S) + 0.5;
  return n > 1.0 ? n : 1.0;
}
// bf16, head dimension 128.  Blocks of 64 rows take two tiles an iteration (0.9 us; 1.1 when two blocks share the keys),
// blocks of 128 one (0.88 us; 0.52 with a single live row group, whose partials are 16 rows).  slots: units of 128 rows that
// the workspace holds.
inline AttnShape plan_bf16_128(int B, int H, int max_nodes, int kv_cap, long long slots, bool two_bf16) {
  AttnShape best = {1, 1};
  const long long bh = (long long)B * H;
  double least = 1e30;
  for (int QB = 1; QB <= (max_nodes > 64 ? 2 : 1); ++QB) {
    const bool rows64 = max_nodes > 64 ? QB == 2 : max_nodes > kFewRows;
    const double iter = rows64 ? (QB == 2 ? 1.1 : 0.9) : (max_nodes > kFewRows ? 0.88 : 0.52);
    for (int S = 1; S <= kMaxKvSplits; ++S) {
      const long long groups = bh * QB * S;
      if (S > 1 && (groups > 256 || groups > slots || S * 4 > (kv_cap + max_nodes + kTileKeys - 1) / kTileKeys)) break;
      const double us = taking_turns(groups / 256.0, B > 1 ? 0.7 : 1.0) * (4.8 + iterations(kv_cap, max_nodes, S, rows64 ? 2 : 1) * iter) +
                        split_us(bh, S, max_nodes, 128, two_bf16);
      if (us < least) {
        least = us;
        best = {QB, S};
      }
    }
  }
  return best;
}
// Everything else, blocks of 64 rows.  Float: the matrix rate, workgroups on one compute unit take turns as far as their
// wavefronts have rows; bf16: they run side by side.  slots: units of 64 rows.
inline AttnShape plan_any(int B, int H, int max_nodes, int kv_cap, int dh, bool f32, long long slots, bool two_bf16) {
  AttnShape best = {(max_nodes + 63) / 64, 1};
  const long long bh = (long long)B * H, blocks = bh * best.QB;
  const int live = max_nodes >= 64 ? 4 : (max_nodes + 15) / 16;
  double least = 1e30;
  for (int S = 1; S <= kMaxKvSplits; ++S) {
    if (S > 1 && (blocks * S > slots || S * kTileKeys > kv_cap + max_nodes || bh > 65535)) break;  // (the merge's grid)
    const long long groups = blocks * S;
    const double turns = f32 && dh > 32 ? taking_turns((double)((groups * live + 1023) / 1024), B > 1 ? 0.5 : 1.0) : side_by_side(groups / 256.0);
    const double tile = f32 ? (dh <= 16 ? 0.7 : dh <= 32 ? 0.9 : (dh + 31) / 32 * 32 / 48.0) : (dh <= 64 ? 0.6 : 0.7);
    const double us = turns * (3.0 + iterations(kv_cap, max_nodes, S, 1) * tile) + split_us(bh, S, max_nodes, dh, two_bf16);
    if (us < least) {
      least = us;
      best.S = S;
    }
  }
  return best;
}

}  // namespace ctcspec
