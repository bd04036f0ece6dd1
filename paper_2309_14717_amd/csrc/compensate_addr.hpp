// Byte offsets of the loads of U in compensate_kernel (compensate.hip): a buffer resource per block of
// 128 rows, an offset per lane and one per row.  The hardware's range check looks at the lane's offset,
// not at the row's, so the row offsets must not lead out of the block by themselves.
#pragma once
#include "common.hpp"

namespace qalora {

constexpr int kCompBlock = 128;  // rows per lazy block (a multiple of every supported group size)

__host__ __device__ constexpr int comp_block_rows(int d_in, int blk) {
  return d_in - blk * kCompBlock < kCompBlock ? d_in - blk * kCompBlock : kCompBlock;
}

// Updating wavefronts: lane (n, kb) reads NT adjacent elements, from column r0 + NT n, of rows
// 16 k + 4 q + kb of a block.  They only ever read blocks that another one follows (128 rows each);
// in a matrix of one panel they have nothing to do.
__host__ __device__ constexpr bool comp_updates(int panels) { return panels > 1; }
__host__ __device__ constexpr uint32_t comp_update_lane(uint32_t row_b, int nt, int r0, int n, int kb) {
  return (uint32_t)kb * row_b + 4u * (uint32_t)(r0 + nt * n);
}
__host__ __device__ constexpr uint32_t comp_update_row(uint32_t row_b, int k, int q) {
  return (uint32_t)(16 * k + 4 * q) * row_b;
}

// The walker: rows 16 s + 4 q + kb of its panel, which may have fewer rows than that (half a tile
// at the end: no lane reads anything then).
__host__ __device__ constexpr uint32_t comp_walk_row(uint32_t row_b, int rows, int s, int q) {
  return (uint32_t)(16 * s + 4 * q < rows ? 16 * s + 4 * q : rows) * row_b;
}

}  // namespace qalora
