// Launch shapes of the front launch (adapter.hip).
#pragma once
#include <algorithm>

#include "common.hpp"

namespace qalora {

// Columns per block of the factor job: as many (up to 16) as keep its LDS tile of L x columns
// fp32 values within 32 KB, so that the row jobs of the same launch keep their occupancy.
inline int factor_cols(int L) {
  int fc = 16;
  while (fc > 1 && (size_t)L * fc * 4 > 32 * 1024) fc >>= 1;
  return fc;
}

// Up to 1024 rows of a forward beside its factor job, in one launch with it (a launch of their own before it: 2 to 4 us more
// almost everywhere): a block each, or a wavefront?  A wavefront takes a row of up to 4096 elements in one sweep and is
// hidden under the job; longer rows are read twice and end the launch where the job's blocks are short, which is where
// groups are few (L, that is long rows of large groups) and the rank is low.  Blocks of rows in turn delay a long job, more
// so where more than the 1024 blocks that run at once (37 KB of LDS and the registers leave four a unit) come before
// the job's last one.  Fitted to 630 pairs with an adapter (rank 16 to 128, with pooling and without) and 184 without,
// 40 to 1000 tokens of 1024 x 1024 to 13824 x 13824 and 22016 x 8192: 0.2 % from the better one on average, 3.5 % at most (always
// blocks: 0.8 and 12; with an adapter by their number alone, and without one up to 96 rows: 0.8 and 15, 2.2 and 17).  us by
// wavefronts / by blocks: adapter-free, 300 tokens of 13824 x 5120, g 128 83 / 74, g 32 87 / 88; 700 of 8192 x 22016, g 32 339 / 348;
// with pooling, 200 of 13824 x 13824, rank 16 g 128 128 / 112, rank 128 g 32 166 / 181.
inline bool front_rows_by_block(int T, int d_in, int g, int d_out, bool fold, int rank, bool pooled) {
  if (T <= 64) return true;
  const bool one_sweep = d_in <= 4096;
  if (!fold) return one_sweep ? T <= 256 : g >= 64;
  const int job = ceil_div(d_out, factor_cols(d_in / g)), longer = rank + 24;
  const bool at_once = job + std::min(job, T) <= 1024;
  if (one_sweep) return at_once && (pooled || T <= 256) && longer < 4 * g;
  return (pooled ? 3 : 2) * g > (at_once ? longer : 2 * longer);
}

}  // namespace qalora
