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
// A call's time by what it is made of, in us:
//   workgroups a compute unit takes in turn x (start of one + iterations x time of one) + what splitting costs
// Splitting costs the merge launch and the partial results, which go through memory.  Both kernels start from as many
// splits as fill the chip (at most 8, a few tiles each; two blocks of 64 rows where they fill as much) and take the cheapest
// (query blocks, key splits) of the model instead where it spares 3 %.  Measured in HIP graphs, us a call as the chip is filled /
// with this choice:
//   bf16, 128: 2 x 40 heads, 128 rows, 128 positions 17.1 (2 splits) / 10.0 (none, two blocks)    6 x 32 heads, 200: 22.3 / 16.8
//     (one block)    4 x 32 heads, 100 rows, 300: 18.5 (2) / 13.2 (1)    32 heads, 64 rows, 256: 11.9 (2) / 10.2 (1)
//     32 heads, 128 rows, 2048 positions: 4 splits both; none 36.8, 2 26.0, 3 21.6, 4 19.6, 8 of one block 20.0
//   bf16, 80: 4 x 16 heads, 50 rows, 93 positions 10.5 (2) / 7.6 (1)
//   float, 128: 14 heads, 35 rows, up to 1923 positions 24.0 (8) / 18.4 (24)    float, 16: 4 heads, 128 rows, 32: 7.4 (3) / 4.0 (1, padded
//     to 16 instead of 32)
// Every plan of 1460 shapes drawn from 1 to 8 sequences of 4 to 40 heads and 1 to 128 rows over 4 to 2048 positions was timed, and
// the constants are the ones of a coarse grid (the same for both kernels where they mean the same) that come closest to the best
// plan of each: within 1.1 % in the mean (bf16, 128), 1.0 (bf16, others), 1.5 (float) and 1.1 (float heads up to 32); on 510 further
// shapes 0.9, 0.7, 1.1 and 3.2 %.  That is 4.8, 8.3, 5.8 and 5.8 % less than as the chip is filled (further shapes: 4.2, 8.0,
// 5.2 and 7.5); 18 of the 1970 take more than 4 % longer than that, the worst 11 %.
constexpr int kFillSplits = 8;
constexpr double kModelGain = 0.97;
// the merge launch with the end of the kernel before it, whose stores it waits for (behind an independent kernel a launch takes 2.2
// us; with that in its place the mean is 1 % worse), the partial results' way through memory, and a round trip of the merge for every eight
// splits more.  Rows as two bf16 numbers are the merge's work otherwise: the 2 x 8 rows of a layer of 1024, 300 positions, 42.2 us with
// the layer's attention in two splits, 44.0 in none.
constexpr double kMergeUs = 3.5, kTwoBf16Us = 1.5;
inline double split_us(long long bh, int S, int rows, int dh, bool two_bf16) {
  return S == 1 ? (two_bf16 ? kTwoBf16Us : 0.0) : kMergeUs + (double)bh * S * rows * dh * 4 * 0.33e-6 + (S - 1) / kMergeParts * 2.0;
}
// how much longer than one workgroup a compute unit with `load` of them takes.  Of several sequences, not all are the longest.
inline double taking_turns(double load, double next) { return load <= 1.0 ? 1.0 : 1.0 + (load - 1.0) * next; }
// (two at a time hide each other's waits)
inline double side_by_side(double load) { return load <= 1.0 ? 1.0 : load <= 2.0 ? 1.1 + (load - 1.0) * 0.2 : load * 0.68; }
// tiles of 32 keys that a workgroup expects: the lengths are on the device, the host takes the capacity for them;
// what does not divide leaves part of an iteration idle
inline double iterations(int kv_cap, int max_nodes, int S, int per_iter) {
  const double n = (double)(kv_cap + max_nodes) / (kTileKeys * per_iter * S) + 0.4;
  return n > 1.0 ? n : 1.0;
}
// bf16, head dimension 128.  Blocks of 64 rows take two tiles an iteration (0.9 us; 0.95 when two blocks share the keys),
// blocks of 128 one (0.72 us; 0.52 with a single live row group, whose partials are 16 rows), all of them a fifth longer when
// every compute unit has one.  slots: units of 128 rows that the workspace holds.
inline AttnShape plan_bf16_128(int B, int H, int max_nodes, int kv_cap, long long slots, bool two_bf16) {
  const long long bh = (long long)B * H;
  const int key_tiles = (kv_cap + max_nodes + kTileKeys - 1) / kTileKeys;
  auto fill = [&](int QB) {
    long long S = 256 / (bh * QB);
    S = S > key_tiles / 4 ? key_tiles / 4 : S;
    S = S > kFillSplits ? kFillSplits : S;
    while (S > 1 && bh * QB * S > slots) --S;
    return S < 1 ? 1 : (int)S;
  };
  auto us_of = [&](AttnShape s) {
    const bool rows64 = attn_rows64(s, max_nodes);
    const double iter = rows64 ? (s.QB == 2 ? 0.95 : 0.9) : (max_nodes > kFewRows ? 0.72 : 0.52);
    const double load = (double)(bh * s.QB * s.S) / 256.0;
    return taking_turns(load, B > 1 ? 1.5 : 1.0) * (1.0 + 0.2 * (load < 1.0 ? load : 1.0)) *
               (8.0 + iterations(kv_cap, max_nodes, s.S, rows64 ? 2 : 1) * iter) +
           split_us(bh, s.S, max_nodes, 128, two_bf16);
  };
  const int s128 = fill(1), s64 = fill(2);
  AttnShape best = {1, s128};
  if (max_nodes > 64 && (2 * s64 > s128 || (2 * s64 == s128 && s64 >= 4))) best = {2, s64};
  double least = kModelGain * us_of(best);
  for (int QB = 1; QB <= (max_nodes > 64 ? 2 : 1); ++QB) {
    for (int S = 1; S <= kMaxKvSplits; ++S) {
      const long long groups = bh * QB * S;
      if (S > 1 && (groups > 256 || groups > slots || S * 4 > key_tiles)) break;
      const double us = us_of({QB, S});
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
  const int QB = (max_nodes + 63) / 64, live = max_nodes >= 64 ? 4 : (max_nodes + 15) / 16;
  const long long bh = (long long)B * H, blocks = bh * QB;
  if (bh > 65535) return {QB, 1};  // (the merge's grid)
  auto us_of = [&](int S) {
    const long long groups = blocks * S;
    const double turns = f32 && dh > 32 ? taking_turns((double)((groups * live + 1023) / 1024), B > 1 ? 0.35 : 1.0) : side_by_side((double)groups / 256.0);
    const double tile = f32 ? (dh <= 16 ? 0.6 : dh <= 32 ? 0.9 : (dh + 31) / 32 * 32 / 48.0) : (dh <= 64 ? 0.6 : 0.7);
    return turns * (3.0 + iterations(kv_cap, max_nodes, S, 1) * tile) + split_us(bh, S, max_nodes, dh, two_bf16);
  };
  long long fill = 512 / blocks;  // two workgroups per compute unit, two tiles each
  const int key_tiles = (kv_cap + max_nodes + kTileKeys - 1) / kTileKeys;
  fill = fill > key_tiles / 2 ? key_tiles / 2 : fill;
  fill = fill > kFillSplits ? kFillSplits : fill;
  while (fill > 1 && blocks * fill > slots) --fill;
  AttnShape best = {QB, fill < 1 ? 1 : (int)fill};
  double least = kModelGain * us_of(best.S);
  for (int S = 1; S <= kMaxKvSplits; ++S) {
    if (S > 1 && (blocks * S > slots || S * kTileKeys > kv_cap + max_nodes)) break;
    const double us = us_of(S);
    if (us < least) {
      least = us;
      best.S = S;
    }
  }
  return best;
}

}  // namespace ctcspec
