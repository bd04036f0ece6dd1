// Launch shape of the dequantising product (gemm_dq.hip).
#pragma once
#include <algorithm>

#include "common.hpp"

namespace qalora {

constexpr int kGemmStep = 64;  // K values per step
constexpr int kGemmMaxSplits = 16;
constexpr size_t kGemmPartialRoom = 256ull << 20;
constexpr size_t kGemmFastPartialRoom = 64ull << 20;  // a 256 x 256 fp32 tile per compute unit

// What the fast addressing path of gemm_dq_kernel needs besides padded activation copies.
inline bool gemm_fast_shape(int K_main, int group) {
  return K_main % kGemmStep == 0 && (kGemmStep % group == 0 || group % kGemmStep == 0);
}

struct GemmPlan {
  int tile_rows;  // 64, 128, 192 or 256
  int ksplit;     // slices of K
};

// What the slices' copies of the output may take (the fast form's; or either's).
inline size_t gemm_dq_partial_room(int M, int N, bool fast = false) {
  return std::min((size_t)kGemmMaxSplits * M * N * 4, fast ? kGemmFastPartialRoom : kGemmPartialRoom);
}

// Tile rows and K splits of the dequantising product, searched together: a launch takes
// rounds(tiles x splits) x (K steps per block + prologue and epilogue), and a split adds the sum over the
// slices (its launch, `splits` fp32 copies of the output written and read again).  A step of a small tile
// costs more per row -- the producer dequantises the same 256 x 64 weights whatever the tile's height -- but
// while compute units are idle that costs nothing, and its blocks start and end sooner: 64-row tiles run
// one or two per unit.  Constants (us) fitted to 484 sweeps over tile and split (16 .. 4096 tokens,
// 512 .. 22016 features, 2 to 4 bits, both directions): the plan is 0.7 % from the best of each sweep on
// average; heights and splits planned one after the other, with at least eight steps per slice, were 13 %
// from it (per call of 512 tokens: 1024 x 4096 38.6 -> 24.5 us, 2048 x 2048 36.9 -> 31.1, 4096 x 4096 48.9 -> 44.6;
// 1024 tokens of 4096 x 4096 71.3 -> 62.2).
// The general form (offsets of every load worked out per step) goes by the same constants but for two (us before / with
// these): its forward's 64-row step is longer (300 tokens of 4800 x 11008, g 96 88 / 70; 512 of 3072 x 4096 41 / 37), and
// its 3-bit backward has one such block on a unit, not two (130 tokens, 13824 x 2720 58 / 52, 11008 x 4072 65 / 60; 107
// sizes of it 0.6 % shorter on average, none longer).  The backward takes it where d_out is no multiple of 64.
// The fast form's slices may take 64 MB: units without a tile give their power to the others, so larger outputs lose by
// slices (90 sweeps of 350 .. 914 tokens: 10 % slower in slices that take more; 914 tokens of 22016 -> 8192 backward 355 us
// whole, 405 in two).  The general form, further from the power limit, gains by them up to 256 MB (147 sweeps of 350 .. 2700
// tokens: 0.4 % from the best on average, 10 % at most; within 64 MB 2.6 and 30; 3-bit backward of 1056 tokens, 9088 x 13480
// 524 / 412).
inline GemmPlan gemm_dq_plan(int bits, int M, int N, int K_main, int group, bool bwd = false) {
  struct Tile {
    int rows;
    double step, block;  // of a K step and of a block's prologue and epilogue
  };
  constexpr Tile kTiles[4] = {{64, 0.63, 1.0}, {128, 0.73, 4.0}, {192, 0.89, 6.1}, {256, 1.05, 8.1}};
  constexpr double kPairStep = 0.98, kPairBlock = 2.0;  // two 64-row blocks on every unit
  constexpr double kClock = 0.1;       // of a round's time that its idle units give back (power)
  constexpr int kUnits = 256;
  const bool fast = gemm_fast_shape(K_main, group);
  const bool single = !fast && bits == 3 && bwd;  // one 64-row block per unit (gemm_min_waves)
  const double bits_step = single ? 1.5 : (bits == 3 ? 1.28 : 1.0);  // two planes to put together
  const int nk = ceil_div(K_main, kGemmStep);
  const double out_us = (double)M * N * 1e-6;
  const size_t room = gemm_dq_partial_room(M, N, fast);
  GemmPlan best{};
  double best_cost = 0;
  for (const Tile& t : kTiles) {
    if (!fast && t.rows > 128) break;  // (the general form is built for the two small tiles)
    if (t.rows > 64 && t.rows - 64 >= M) break;
    const long tiles = (long)ceil_div(M, t.rows) * ceil_div(N, 256);
    for (int ks = 1; ks <= kGemmMaxSplits && ks <= nk; ++ks) {
      if (ks > 1 && (size_t)ks * M * N * 4 > room) break;
      const int steps = ceil_div(nk, ks);
      if (ceil_div(nk, steps) != ks) continue;  // a slice would be empty
      const long blocks = tiles * ks;
      const double one = steps * (t.rows == 64 && !fast && !bwd ? 0.665 : t.step) * bits_step + t.block;
      double cost;
      if (t.rows == 64 && !single) {
        const double pair = steps * kPairStep * bits_step + kPairBlock;
        const long rounds = blocks / (2 * kUnits), rest = blocks - rounds * 2 * kUnits;
        cost = rounds * pair + (rest > kUnits ? pair : (rest > 0 ? one : 0.0));
      } else {
        const long rounds = blocks / kUnits, rest = blocks - rounds * kUnits;
        cost = rounds * one + (rest > 0 ? one * (1.0 - kClock * (1.0 - (double)rest / kUnits)) : 0.0);
      }
      if (ks > 1) {
        cost += 3.0 + 0.34 * ks + out_us * (0.73 * ks + 0.6);
        const double bytes = 4.0 * ks * M * N;  // (beyond some 64 MB not all of them stay in the last-level cache)
        if (bytes > kGemmFastPartialRoom) cost += 0.9 / 4e6 * (bytes - kGemmFastPartialRoom);
      }
      if (best.tile_rows == 0 || cost < best_cost) {
        best = GemmPlan{t.rows, ks};
        best_cost = cost;
      }
    }
  }
  return best;
}

inline size_t gemm_dq_partials(const GemmPlan& p, int M, int N) { return p.ksplit > 1 ? (size_t)p.ksplit * M * N * 4 : 0; }

// ... for any batch of up to M tokens, which is what a workspace has room for.  Batches that have the same tiles get the
// fewer slices the longer they are (a slice's cost grows with the tokens, a step's does not), so the slices at either end
// of a range of them bound what is between.
inline size_t gemm_dq_most_partials(int bits, int M, int N, int K_main, int group, bool bwd) {
  size_t most = 0;
  auto slices = [&](int m) { return gemm_dq_plan(bits, m, N, K_main, group, bwd).ksplit; };
  auto room = [&](int m) { return gemm_dq_partial_room(m, N, gemm_fast_shape(K_main, group)); };
  auto bytes = [&](int ks, int m) { return ks > 1 ? std::min((size_t)ks * m * N * 4, room(m)) : 0; };
  for (int last = M; last > 0 && room(last) > most; last = (last - 1) / 64 * 64) {
    int lo = (last - 1) / 64 * 64 + 1, ks = slices(lo);  // every tile is whole 64-row ones
    while (lo <= last && bytes(ks, last) > most) {  // runs of batches with as many slices
      int same = lo, more = last + 1;
      for (int step = more - same; step > 1; step = more - same) {
        const int mid = same + step / 2;
        (slices(mid) == ks ? same : more) = mid;
      }
      most = std::max(most, bytes(ks, same));
      lo = more;
      if (lo <= last) ks = slices(lo);
    }
  }
  return most;
}

}  // namespace qalora
