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

// Few rows of a forward beside its factor job, in one launch with it (a launch of their own before it: 2 to 4 us more
// almost everywhere): a block each, or a wavefront?  Blocks of rows alternate with the job's, and those that fold an
// adapter are long: where more than the 1024 that run at once (37 KB of LDS and the registers leave four a unit) come
// before the job's last one, a second round of it follows the rows.  Forward and backward, us by wavefronts / by blocks,
// rank 64 to 128: 13824 x 13824, 128 tokens 373 / 367, 200 451 / 461, 640 838 / 869; 5120 x 13824, 200 186 / 185, 640
// 293 / 298; 11008 x 4096, 300 164 / 160, 640 212 / 206; 13824 x 5120 (rank 16), 512 252 / 245.  Without pooling a
// wavefront does less: 4096 x 4096, 200 tokens 75 / 75, 512 113 / 115.  Adapter-free the job is short, and a wavefront a
// row does as well from about a hundred on: 22016 x 8192, 65 tokens 92 / 91, 400 207 / 208, 800 350 / 358;
// 8192 x 22016, 640 281 / 290; 13824 x 5120, 100 50 / 52.
inline bool front_rows_by_block(int T, bool fold, bool pooled, int L, int d_out) {
  if (!fold) return T <= 96;
  const int job = ceil_div(d_out, factor_cols(L));
  return job + std::min(job, T) <= 1024 && (pooled || T <= 256);
}

}  // namespace qalora
