// Launch shape of the mid-token forward (midt.hip).
#pragma once
#include "common.hpp"
#include "kernels.hpp"

namespace qalora {

constexpr int MT_SLAB = 128;  // columns per block: two wavefronts of 64
constexpr int MT_DEEP = 4;    // chunks of 128 rows per unit, one per pair of wavefronts

inline int midt_tiles(int tokens) { return tokens <= 32 ? 2 : (tokens <= 48 ? 3 : 4); }

// Time of a launch on `nb` blocks, less what every launch takes, in a scale of its own (a unit of one token
// tile is 1.2).  More blocks shorten the runs but cut the slabs into more parts, whose sums the block that
// finishes a slab adds.  Fitted to sweeps over the count (1024 .. 22016 features, even and odd widths, 8 to
// 64 tokens, all layouts; 1.3 % from the best count on average):
//   * runs of whole slabs meet no others;
//   * nb a multiple of the slabs: no run crosses a slab, a hand-over each.  One less where only the last part of
//     a slab is longer than the others: they are done before it needs their sums (64 tokens, 2048 x 8192 =
//     64 slabs of 4 units: 18.2 us on 192 blocks, 18.9 on 248, 19.7 on 128);
//   * otherwise runs cross slabs and a block has two sums to deal with;
//   * more on all or nearly all compute units, unless the runs are long (why was not found; 64 tokens,
//     4096 x 4096: 19.3 on 224, 20.2 on 248, 22.6 on 255 and 256; 8192 x 4096: 23.4 on 224, 26.8 on 248;
//     22016 x 8192: 53.4 on 224, 49.8 on 256).
// The best count that fits may cost this much of the best with any room.  (4 bits: deployed layers take the
// same path as triples, and their dense call has no factor pass; 3 bits, 27 tokens of 1280 x 5024: 16.4 us
// at 1.2, 21.5 on the dense kernel.)
inline double midt_short_of(int bits) { return bits == 4 ? 1.15 : 1.5; }
// (3 bits: two code words to put together; 64 tokens, 8192 x 8192 on 64 blocks 67 us against 52 and 53)
inline double midt_unit(int bits, int tt) { return (1.0 + 0.2 * tt) * (bits == 3 ? 1.35 : 1.0); }
inline double midt_least_handover(int tt) { return 0.9 + 0.4 * tt; }
inline bool midt_whole_slabs(int CU, int S, int nb) { return CU == 1 || (nb <= S && S % nb == 0); }
inline double midt_cost(int units, int CU, int S, double unit, int tt, int nb, int parts) {  // parts = ceil(nb / S)
  const int run = (units + nb - 1) / nb, n = parts - 1;
  if (midt_whole_slabs(CU, S, nb)) return run * unit + 0.3;
  if (nb == S * parts)
    return run * unit + 1.6 + 0.4 * tt + 0.3 * n - (CU % parts == 1 ? 1.0 : 0.0) + (nb > 248 ? 0.2 * n : 0.0);
  return 0.5 * (run + (double)units / nb) * unit + 2.5 + 0.5 * tt + 0.3 * n +
         (nb > 248 && units < 6 * 256 ? 2.3 : 0.0);
}

// Blocks of the launch, at most one per compute unit, given the room for flags (ST_HEAD_BYTES) and partials
// behind them (runs of whole slabs need none).  0 where the room leaves too few: the dense kernel is for
// these (none where the room is midt_room).
// Runs on every call, so it ends early: it goes from the most blocks down, and once the units alone cost more
// than the best so far (or than is allowed above the cheapest) fewer blocks only do more each.
inline int midt_blocks(int bits, int d_in, int d_out, int tokens, size_t scratch) {
  const int CU = ceil_div(d_in / 128, MT_DEEP), S = ceil_div(d_out, MT_SLAB);
  if ((long)S * CU > (1l << 22)) return 0;
  const int units = S * CU, tt = midt_tiles(tokens);
  const long room = scratch <= ST_HEAD_BYTES ? 0 : (long)((scratch - ST_HEAD_BYTES) / ((size_t)tt * 4 * 128 * 16));
  const double unit = midt_unit(bits, tt);
  int best = 0;
  double best_cost = 0, free_cost = 0;  // with the room there is, and with any
  const int most = units < ST_MAX_BLOCKS ? units : ST_MAX_BLOCKS;
  int parts = ceil_div(most, S);  // per slab, about
  for (int nb = most; nb >= 1; --nb) {
    if (nb <= S * (parts - 1)) --parts;
    if (free_cost > 0) {
      const double limit = (best > 0 ? best_cost : midt_short_of(bits) * free_cost) * nb * 1.000001;
      if (units * unit > limit) break;
      if (nb > S && CU > 1 && units * unit + midt_least_handover(tt) * nb > limit) {  // on to the whole slabs
        nb = S + 1;
        parts = 2;
        continue;
      }
    }
    const double cost = midt_cost(units, CU, S, unit, tt, nb, parts);
    if (free_cost == 0 || cost < free_cost) free_cost = cost;
    if ((midt_whole_slabs(CU, S, nb) || nb <= room) && (best == 0 || cost <= best_cost)) {
      best = nb;
      best_cost = cost;
    }
  }
  return best > 0 && best_cost <= midt_short_of(bits) * free_cost ? best : 0;
}

// Room that holds the partials of any count for up to so many tokens; 8.4 MB at most.
inline size_t midt_room(int d_in, int d_out, int tokens) {
  const long units = (long)ceil_div(d_in / 128, MT_DEEP) * ceil_div(d_out, MT_SLAB);
  const size_t blocks = units < ST_MAX_BLOCKS ? (size_t)units : (size_t)ST_MAX_BLOCKS;
  return ST_HEAD_BYTES + blocks * midt_tiles(tokens < MT_MAX_TOKENS ? tokens : MT_MAX_TOKENS) * 4 * 128 * 16;
}

}  // namespace qalora
