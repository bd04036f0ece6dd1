// Sums over copies of a matrix, copies in order.
#pragma once
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace qalora {

// v[q] = src[q][0] + src[q][stride] + ... over n copies; the loads of up to B (4 to 8) copies are in flight together
template <int B, int Q>
__device__ __forceinline__ void sum_slices(const f32x4* const (&src)[Q], size_t stride, int n, f32x4 (&v)[Q]) {
#pragma unroll
  for (int q = 0; q < Q; ++q) v[q] = src[q][0];
  auto add = [&](auto n_c, int z0) {
    constexpr int c = decltype(n_c)::value;
    f32x4 ld[c][Q];
#pragma unroll
    for (int z = 0; z < c; ++z)
#pragma unroll
      for (int q = 0; q < Q; ++q) ld[z][q] = src[q][(size_t)(z0 + z) * stride];
#pragma unroll
    for (int z = 0; z < c; ++z)
#pragma unroll
      for (int q = 0; q < Q; ++q) v[q] += ld[z][q];
  };
  int z = 1;
  for (; z + B <= n; z += B) add(std::integral_constant<int, B>{}, z);
  switch (n - z) {  // fewer than B: in flight together as well
    case 7: if constexpr (B > 7) add(std::integral_constant<int, 7>{}, z); break;
    case 6: if constexpr (B > 6) add(std::integral_constant<int, 6>{}, z); break;
    case 5: if constexpr (B > 5) add(std::integral_constant<int, 5>{}, z); break;
    case 4: if constexpr (B > 4) add(std::integral_constant<int, 4>{}, z); break;
    case 3: add(std::integral_constant<int, 3>{}, z); break;
    case 2: add(std::integral_constant<int, 2>{}, z); break;
    case 1: add(std::integral_constant<int, 1>{}, z); break;
    default: break;
  }
}
template <int B = 8>
__device__ __forceinline__ f32x4 sum_slices(const f32x4* src, size_t stride, int n) {
  const f32x4* s[1] = {src};
  f32x4 v[1];
  sum_slices<B>(s, stride, n, v);
  return v[0];
}

// Four elements of the sum over the slices of a split product, converted on the way out.  Bound by the slices'
// bytes where there are enough threads: each then loads slice after slice, since with all slices of a thread in
// flight at once the chip reads from more places than it can keep open (8 slices of 256 x 8192, 67 MB: 11.3 us
// one by one, 12.0 together; 1000 x 4096 11.4 and 11.8).  Few threads wait for one load after the other, and
// there it is the other way round (100 x 1024: 2.7 and 2.2 us); 128 x 4096, where the line lies, takes 4.1 us
// either way.
constexpr size_t kSumOneByOne = 128 * 1024;  // threads: two wavefronts on every SIMD
__device__ __forceinline__ void split_sum_one(const SplitSum& s, size_t i) {
  const f32x4* src = reinterpret_cast<const f32x4*>(s.partial) + i;
  f32x4 v;
  if (s.n4 >= kSumOneByOne) {
    v = src[0];
    for (int z = 1; z < s.slices; ++z) v += src[(size_t)z * s.n4];
  } else {
    v = sum_slices(src, s.n4, s.slices);
  }
  if (s.out_bf16)
    reinterpret_cast<uint2*>(s.out)[i] = uint2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
  else
    reinterpret_cast<f32x4*>(s.out)[i] = v;
}

}  // namespace qalora
