// Launch shapes of the adapters' gradients (grads.hip).
#pragma once
#include <algorithm>

#include "common.hpp"

namespace qalora {

constexpr int MAX_PARTS = 4;  // linears that share their input
constexpr int GZ_L = 128;  // groups per tile
constexpr int GZ_C = 128;  // columns per tile of z_kernel and db_kernel
constexpr int GZ_T = 64;   // tokens per step of theirs
constexpr int GF_C = 32;   // columns per block of finish_kernel and fused_kernel
constexpr int GA_T = 32;   // tokens per step of a dA block
constexpr int kGradsFusedTokens = 640, kGradsShort = 128;
constexpr int kGradsDuSlices = 24;  // partial sums of dU, at most

// Equal runs of units (a tile's step of tokens), tile by tile.
struct ZRuns {
  int steps, units, blocks;  // of a tile; in all; one run each
  __host__ __device__ int first(int b) const { return (int)((long)b * units / blocks); }            // unit of block b
  __host__ __device__ int owner(int u) const { return (int)(((long)(u + 1) * blocks - 1) / units); }  // block of unit u
};
enum GradsForm { GRADS_FUSED, GRADS_BY_Z, GRADS_BY_U };
struct GradsPlan {
  GradsForm form;
  ZRuns runs;  // by Z: of its tiles; by U: of dB's
  int slots;   // partial sums of a tile, at most
  // by U
  int rank_tile;                             // 32, 64 or 128
  int tile0[MAX_PARTS];                      // first tile of a part
  bool du_long;                              // dU in blocks of 256 tokens
  int du_steps, du_slices[MAX_PARTS];        // steps of 64 columns in a partial sum of dU, and partial sums
  int da_tokens, da_shares;                  // tokens in a share of dA, and shares
};
// fused and by Z: shares of dA that a part of so many columns leaves; of dB that so many groups leave (0: it comes out
// whole)
inline int grads_da_shares(int d_out) { return ceil_div(d_out, GF_C); }
inline int grads_db_shares(int L) { return L <= GZ_L ? 0 : ceil_div(L, GZ_L); }

// Which form.
// Fused: few tokens and no more blocks than compute units (forward and backward of 64 tokens, 1024 x 1024 rank
// 16: 37.7 us against 42.1 with two; 512 of 4096 x 4096 rank 64: 107 / 112; 1024 of 2048 x 2048: 86.9 / 85.1; 128 of
// 4096 x 11008, 344 blocks: 108.6 / 106.5; 128 groups by four wavefronts, eight are 1 to 8 % of the step faster).
// Else by Z or by U, whichever a linear model says is shorter: Z makes T d_out L products and L r d_out fp32 ones, with
// shares of dA to every 32 columns; U two times T d_out r (tiles of 32, 64, 128), and reads dy twice.  Coefficients (us) fitted
// to 490 pairs (40 to 4096 tokens, 32 to 432 groups, ranks 16 to 128, 2048 to 22016 columns): the choice costs 0.3 % of the
// gradients' launches on average and 0.1 % of the step, 9 % of one at most (short batches, where launches by U are chains of
// waits).  The gradients and the conversion of dy, Z / U in us: 4096 tokens of 4096 x 4096 rank 64 48 / 51, of 11008 x 4096 79 / 59;
// 1531 of 5120 x 13824 g 64 rank 64 60.7 / 65.8; 700 of 4096 x 4096 rank 16 29.6 / 24.8; 4096 of 4096 x 22016 rank 64
// 168 / 178, rank 16 160 / 143.
inline int grads_group_tile(int L) { return L <= 32 ? 32 : (L <= 64 ? 64 : GZ_L); }  // rows of a tile of Z
inline bool grads_fusable(int L, int d_out) { return ceil_div(d_out, GF_C) * ceil_div(L, GZ_L) <= 256; }
inline GradsForm grads_form(int T, int L, int d_out, int max_rank, int rank_tile) {
  if (T <= kGradsFusedTokens && grads_fusable(L, d_out)) return GRADS_FUSED;
  const double l_tiles = grads_group_tile(L) * ceil_div(L, GZ_L), tokens = round_up(T, GZ_T), n = d_out;
  const double z_less_u = -3.26 + 1e-9 * tokens * n * (4.2 * L - 16.9 * rank_tile + 378.0) + 46.5e-9 * n * L * max_rank +
                          n * (5.11e-6 * l_tiles - 6.15e-6 * rank_tile) - (T <= kGradsShort ? 2.17 : 0.0);
  return z_less_u > 0 ? GRADS_BY_U : GRADS_BY_Z;
}

// By U: rows of dU's partial sums, and shares of dA, that no plan of up to T tokens exceeds.
inline size_t grads_most_du_rows(int T) { return std::min<size_t>((size_t)kGradsDuSlices * T, std::max(65536, T)); }
// (a block of dA takes as long as it has tokens: 4096 tokens of 4096 x 4096 rank 64, 32 shares 30.8 us with dB, 128 16.9)
inline int grads_most_da_shares(int T, int L, int n_parts) {
  return std::min(ceil_div(T, GA_T), std::min(128, std::max(16, 256 / (ceil_div(L, GZ_L) * n_parts))));
}

// Runs of z_kernel and db_kernel: a block per compute unit, two where the runs are long: two cover each other's waits, but
// leave twice as many partial sums.  For Z from 3000 units on (two against one, 216 calls: 4 % longer below 3000, 2 to 3 %
// shorter to 6000, 8 above; 4096 tokens of 5120 x 13824 g 64 116 us against 122), for dB from 8192 (with dA's blocks beside them:
// 2 to 6 % longer below).
// dU: blocks of 64 tokens up to 1024, else of 256 (4096 tokens of 4096 x 22016 rank 64: 72 us in blocks of 64, 63 in
// those; 1024 of 4096 x 4096 9.7 / 10.3), and as many partial sums as fill the chip, up to 24 or 16: dA's blocks add
// them (20 tokens of 13824 x 13824 rank 128: 29 us with 16, 20 with 24).
// (`form`: where given, that one)
inline GradsPlan grads_plan(int T, int L, int d_out, int n_parts, const int* rank, const int* part_dout,
                            const GradsForm* form = nullptr) {
  GradsPlan p{};
  const int steps = ceil_div(T, GZ_T);
  auto in_runs = [&](int tiles, long most_for_one) {
    const long units = (long)steps * tiles;
    p.runs.steps = steps;
    p.runs.units = (int)units;
    p.runs.blocks = (int)std::min(units, units > most_for_one ? 512L : 256L);
    p.slots = std::min(steps, ceil_div(p.runs.blocks, tiles) + 1);
  };
  int max_rank = 0, tiles = 0, all = 0;
  for (int q = 0; q < n_parts; ++q) {
    max_rank = std::max(max_rank, rank[q]);
    p.tile0[q] = tiles;
    tiles += ceil_div(part_dout[q], GZ_C);
    all += ceil_div(part_dout[q], 64);
  }
  p.rank_tile = max_rank <= 32 ? 32 : (max_rank <= 64 ? 64 : 128);
  p.form = form ? *form : grads_form(T, L, d_out, max_rank, p.rank_tile);
  if (p.form == GRADS_BY_Z) in_runs(ceil_div(d_out, GZ_C) * ceil_div(L, GZ_L), 3000);
  if (p.form != GRADS_BY_U) return p;
  in_runs(tiles, 8192);
  p.du_long = T > 1024;
  const int most = p.du_long ? 16 : kGradsDuSlices;
  const int slices = std::max(1, std::min(most, p.du_long ? 256 / ceil_div(T, 256) : 512 / ceil_div(T, 64)));
  p.du_steps = ceil_div(all, slices);
  for (int q = 0; q < n_parts; ++q) p.du_steps = std::max(p.du_steps, ceil_div(ceil_div(part_dout[q], 64), most));
  for (int q = 0; q < n_parts; ++q) p.du_slices[q] = ceil_div(ceil_div(part_dout[q], 64), p.du_steps);
  p.da_tokens = GA_T * ceil_div(T, grads_most_da_shares(T, L, n_parts) * GA_T);
  p.da_shares = ceil_div(T, p.da_tokens);
  return p;
}

}  // namespace qalora
