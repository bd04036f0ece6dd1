// Launch shape of the mid-token forward (midt.hip).
#pragma once
#include "common.hpp"
#include "kernels.hpp"

namespace qalora {

constexpr int MT_SLAB = 128;  // columns per block: two wavefronts of 64
constexpr int MT_DEEP = 4;    // chunks of 128 rows per unit, one per pair of wavefronts

inline int midt_tiles(int tokens) { return tokens <= 32 ? 2 : (tokens <= 48 ? 3 : 4); }

// Blocks of the launch, at most one per compute unit, given the room for flags (ST_HEAD_BYTES) and partials
// behind them.  More blocks shorten the runs but cut the slabs into more parts, whose sums the block that
// finishes a slab adds.  Priced in us, fitted to sweeps over the count: a unit 1 + 0.35 per token tile, a
// hand-over 2 and 0.2 per part, runs that end inside a slab 1.5 (a second flush), and 2.3 for more than 31
// blocks per XCD unless the runs are long (the cause of that step was not found; 64 tokens, 4096 x 4096:
// 20.3 us on 128 blocks, 19.5 on 224, 20.2 on 248, 22.6 on 255 and 256; 5120 x 13824: 28.5 on 216 = two per
// slab, 30.1 on 248; 22016 x 8192: 53.4 on 224, 49.8 on 256).  Runs of whole slabs need no room.  0 where the
// best that fits costs a quarter more than the best with any room: the dense kernel is for these.
// Runs on every call, so it ends early: from the most blocks down, a count whose units alone cost more than
// the best so far (or than a quarter above the cheapest) ends the search, since fewer blocks only do
// more each.
inline int midt_blocks(int d_in, int d_out, int tokens, size_t scratch) {
  const int CU = ceil_div(d_in / 128, MT_DEEP), S = ceil_div(d_out, MT_SLAB);
  if ((long)S * CU > (1l << 22)) return 0;
  const int units = S * CU, tt = midt_tiles(tokens);
  const long room = scratch <= ST_HEAD_BYTES ? 0 : (long)((scratch - ST_HEAD_BYTES) / ((size_t)tt * 4 * 128 * 16));
  const double unit_cost = 1.0 + 0.35 * tt;
  int best = 0;
  double best_cost = 0, free_cost = 0;  // with the room there is, and with any
  const int most = units < ST_MAX_BLOCKS ? units : ST_MAX_BLOCKS;
  int parts = ceil_div(most, S);  // per slab, about
  for (int nb = most; nb >= 1; --nb) {
    if (nb <= S * (parts - 1)) --parts;
    const double share = (double)units / nb;
    if (share * unit_cost > (best > 0 ? best_cost : 1.25 * free_cost) && free_cost > 0) break;
    const int run = (units + nb - 1) / nb;
    const bool even = run * nb == units;
    const bool whole = even && run % CU == 0;                         // runs of whole slabs
    const bool inside = CU == 1 || whole || (even && CU % run == 0);  // no run goes on into another slab
    const int n = whole || CU == 1 ? 0 : parts - 1 + !inside;  // sums to wait for, about
    const double cost = (inside ? (double)run : share) * unit_cost + (n > 0 ? 2.0 + 0.2 * n : 0.0) + (inside ? 0.0 : 1.5) +
                        (nb > 248 && units < 6 * 256 ? 2.3 : 0.0);
    if (free_cost == 0 || cost < free_cost) free_cost = cost;
    if ((whole || CU == 1 || nb <= room) && (best == 0 || cost <= best_cost)) {
      best = nb;
      best_cost = cost;
    }
  }
  return best > 0 && best_cost <= 1.25 * free_cost ? best : 0;
}

}  // namespace qalora
