// draft_layer_forward: how the passes over the weight matrices are cut up, and the workspace that takes.  Host code without
// HIP, so that a test can ask it which shapes a call takes.
#pragma once

#include <stddef.h>

namespace ctcspec {

constexpr int kLtMaxCols = 64;  // columns of a pass; each is two bf16 columns (high and low part)
constexpr int kLtMaxSplits = 16;
constexpr int kLtTripK = 256;   // k elements of a trip of the tile loop (4 steps of 64): splits are whole trips

struct LayerPlan {
  int N, K, cols;  // out features, in features, columns of the pass
  int splits;      // k splits, each leaving [cols][N] sums
  int rows;        // weight rows of a workgroup
};

inline int tile_columns(int cols) { return cols <= 16 ? 32 : (cols <= 32 ? 64 : 128); }

// Rows of a workgroup and k splits of an [N][K] pass: fewest microseconds by the model
//   rounds over the compute units x (steps x time of a step + 6 us until the first tile is in LDS)
//   + the partial sums written and read back at 5 TB/s,
// a step taking what the compute unit needs for its bytes: 45 GB/s for weights and activations together (1.39 us
// per 64 KB step), 25 GB/s for the weights alone (its share of HBM).  Taken from a tile loop through registers; with the loads straight into
// LDS the choice is still within 1.5 % of the best of all (rows, splits) at the 7B shape.
inline bool make_plan(LayerPlan& pl, int N, int K, int cols, int plane_cols, int cus) {
  if (K % kLtTripK != 0 || N % 16 != 0 || cols < 1 || cols > kLtMaxCols) return false;
  if ((long long)K * 2 * 256 >= (1LL << 32) || (long long)K * 4 * plane_cols >= (1LL << 32)) return false;  // 32-bit offsets
  const int trips = K / kLtTripK, tile_cols = tile_columns(cols);
  double best = 0.0;
  pl.N = N; pl.K = K; pl.cols = cols; pl.splits = 0; pl.rows = 0;
  for (int rows = 128; rows <= 256; rows += 64) {
    if (rows == 192 && tile_cols == 32) continue;  // no such shape
    const int rb = (N + rows - 1) / rows;
    const double step_us = rows * 80.0 > tile_cols * 100.0 ? rows * 128.0 / 25e3 : (rows + tile_cols) * 128.0 / 45e3;
    for (int s = 1; s <= kLtMaxSplits && s <= trips; ++s) {
      const double rounds = (double)(((long long)rb * s + cus - 1) / cus);
      const double us = rounds * (4.0 * ((trips + s - 1) / s) * step_us + 6.0) + (double)s * N * cols * 8.0 / 5e6;
      if (pl.splits == 0 || us < best) {
        best = us;
        pl.splits = s;
        pl.rows = rows;
      }
    }
  }
  return true;
}

// Ranges of two trips, up to 16 columns, weights that are streamed: the tile goes through registers (gemm_tile.h).  All of such a range
// is requested at once by the loop that loads straight into LDS, and it takes longer than the other loop, whose loads follow one
// another.  A pass over an [N][K] matrix through registers / straight into LDS, us: 6144 x 2048 in 4 ranges 7.3 / 7.9, 8192 x 2048 in 4 8.6 to
// 8.9 / 9.4, 2048 x 5632 in 11 7.3 / 7.6, 4096 x 4096 and 4096 x 11008 in 8 together 26.6 / 27.0.  Ranges of one trip: 2048 x 2048 in 8 5.2 / 5.0,
// 3072 x 1024 in 4 (not streamed) 5.1 / 4.3; of more: 11264 x 2048 in 2 11.0 / 11.0, 12288 x 4096 in 2 20.4 / 18.7, 15360 x 5120 in 2 26.4 / 25.5.
inline bool through_registers(const LayerPlan& pl, bool streamed) {
  const int trips = pl.K / kLtTripK;
  return streamed && pl.rows == 128 && tile_columns(pl.cols) == 32 && (trips + pl.splits - 1) / pl.splits == 2;
}

struct LayerWorkspace {
  size_t q, arows, h1, xn2, act, n_rows, causal, ss1, ss2, part, total;
};
// any_smaller: room for the plans of every smaller B*T too - fewer columns may take more splits and more partial sums, and
// a workspace sized for the largest batch has to serve the others.  Within the tile widths (up to 16, 32, 64 columns) the
// model's splits only fall as the columns grow, so the splits at the narrowest of a width, times its columns, are a bound.
inline LayerWorkspace layer_workspace(int B, int T, int D, int H, int F, int cus, bool any_smaller) {
  LayerWorkspace w;
  size_t off = 0;
  auto carve = [&](size_t bytes) { size_t at = off; off = (off + bytes + 255) / 256 * 256; return at; };
  const size_t BT = (size_t)B * T;
  w.q = carve(BT * D * 2); w.arows = carve(BT * D * 4);
  w.h1 = carve(BT * D * 4); w.xn2 = carve(BT * D * 4); w.act = carve(BT * F * 4);
  w.n_rows = carve((size_t)B * 4); w.causal = carve(BT * 8);
  w.ss1 = carve(BT * (D / 256 + 1) * 4); w.ss2 = carve(BT * (D / 256 + 1) * 4);
  size_t max_floats = 0;
  const int shapes[4][2] = {{3 * D, D}, {D, D}, {2 * F, D}, {D, F}};
  const long long most = (long long)BT < kLtMaxCols ? (long long)BT : kLtMaxCols, last = (long long)BT % kLtMaxCols;
  for (auto& s : shapes) {
    auto room = [&](int plan_cols, long long cols) {
      LayerPlan pl;
      if (plan_cols < 1 || !make_plan(pl, s[0], s[1], plan_cols, (int)BT, cus)) return;
      const size_t floats = (size_t)pl.splits * cols * s[0];
      max_floats = floats > max_floats ? floats : max_floats;
    };
    if (any_smaller) {
      for (int widest = 16; widest <= kLtMaxCols; widest *= 2) {
        const int narrowest = widest == 16 ? 1 : widest / 2 + 1;
        if (narrowest <= most) room(narrowest, most < widest ? most : widest);
      }
    } else {  // full passes, and the last one
      room((int)most, most);
      room((int)last, last);
    }
  }
  w.part = carve(max_floats * sizeof(float));
  w.total = off;
  return w;
}

}  // namespace ctcspec
