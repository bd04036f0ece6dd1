// Launch rules of the dequantising product (gemm_dq_impl.hpp), the sum over the slices of a split K range,
// and the plain product of the adapter gradients.
#include "gemm_dq_impl.hpp"

namespace qalora {

// (gemm_dq_192.hip)
hipError_t launch_192(int bits, bool bwd, const GemmArgs& a, int ks, hipStream_t st, hipEvent_t e0, hipEvent_t e1);

template <int NBITS, bool BWD>
static hipError_t launch_dir(const GemmArgs& a, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const int ks = a.ksplit > 1 ? a.ksplit : 1;
  if (a.a_main_padded_rows >= round_up(a.M, 256) && gemm_fast_shape(a.K_main, a.group)) {
    if (a.tile_rows == 256) return launch_cfg<NBITS, BWD, 256, 256, 2, 4, true, true>(a, ks, st, e0, e1);
    if (a.tile_rows == 192) return launch_192(NBITS, BWD, a, ks, st, e0, e1);
    if (a.tile_rows == 128) return launch_cfg<NBITS, BWD, 128, 256, 2, 4, true, true>(a, ks, st, e0, e1);
    return launch_cfg<NBITS, BWD, 64, 256, 1, 8, true, true>(a, ks, st, e0, e1);
  }
  if (a.tile_rows > 64) return launch_cfg<NBITS, BWD, 128, 256, 2, 4, true, false>(a, ks, st, e0, e1);
  return launch_cfg<NBITS, BWD, 64, 256, 1, 8, true, false>(a, ks, st, e0, e1);
}

// out = sum over the K slices of the partial products, slice order, converted on the way out
__global__ __launch_bounds__(256) void split_reduce_kernel(const float* __restrict__ part,
                                                           int nparts, size_t n4, void* out,
                                                           int out_bf16) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;  // group of 4 elements
  if (i >= n4) return;
  const f32x4* src = reinterpret_cast<const f32x4*>(part) + i;
  f32x4 v = src[0];
  auto add = [&](auto n_c, int z0) {  // n slices, their loads in flight together
    constexpr int n = decltype(n_c)::value;
    f32x4 ld[n];
#pragma unroll
    for (int q = 0; q < n; ++q) ld[q] = src[(size_t)(z0 + q) * n4];
#pragma unroll
    for (int q = 0; q < n; ++q) v += ld[q];
  };
  int z = 1;
  for (; z + 4 <= nparts; z += 4) add(std::integral_constant<int, 4>{}, z);
  if (z + 2 <= nparts) add(std::integral_constant<int, 2>{}, z), z += 2;
  if (z < nparts) add(std::integral_constant<int, 1>{}, z);
  if (out_bf16)
    reinterpret_cast<uint2*>(out)[i] = uint2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
  else
    reinterpret_cast<f32x4*>(out)[i] = v;
}

ProfileHook g_profile_hook[2] = {{nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr}};

static hipError_t launch_bits(int bits, bool bwd, const GemmArgs& a, hipStream_t st, hipEvent_t e0,
                              hipEvent_t e1) {
  if (bits == 4) return bwd ? launch_dir<4, true>(a, st, e0, e1) : launch_dir<4, false>(a, st, e0, e1);
  if (bits == 3) return bwd ? launch_dir<3, true>(a, st, e0, e1) : launch_dir<3, false>(a, st, e0, e1);
  return bwd ? launch_dir<2, true>(a, st, e0, e1) : launch_dir<2, false>(a, st, e0, e1);
}

hipError_t launch_gemm_dq(int bits, bool bwd, const GemmArgs& args, hipStream_t st) {
  GemmArgs a = args;
  const bool split = a.ksplit > 1;
  if (split) {  // slices write fp32 partials; the sum is converted afterwards
    a.out = a.partial;
    a.out_bf16 = 0;
  }
  ProfileHook hook = g_profile_hook[bwd ? 1 : 0];
  g_profile_hook[bwd ? 1 : 0] = ProfileHook{nullptr, nullptr, nullptr, nullptr, 0};
  a.clock_probe = hook.clock_probe;
  a.block_times = hook.block_times;
  a.block_times_cap = hook.block_times_cap;
  // without a split the events ride on the dispatch itself; with one they bracket both launches
  const bool ride = !split && hook.start && hook.stop;
  if (hook.start && !ride) (void)hipEventRecord(hook.start, st);
  hipError_t e = launch_bits(bits, bwd, a, st, ride ? hook.start : nullptr, ride ? hook.stop : nullptr);
  if (e == hipSuccess && split) {
    const size_t n4 = (size_t)a.M * a.N / 4;  // N is a multiple of 8
    split_reduce_kernel<<<(unsigned)((n4 + 255) / 256), 256, 0, st>>>(a.partial, a.ksplit, n4,
                                                                      args.out, args.out_bf16);
    e = hipGetLastError();
  }
  if (hook.stop && !ride) (void)hipEventRecord(hook.stop, st);
  return e;
}

// Plain bf16 x bf16^T product  out[z][M][N] = a_tail[M, Kz] . b_tail[N, Kz]^T  with the K
// range split over `ksplit` slices (partial sums, reduced by the caller in a fixed order).
// Row tile of the plain product by its K length: 128 rows from 128 K steps on (measured: the
// dU product of a layer with D_out = 11008 runs 35 -> 24 us on the taller tile, the one with
// D_out = 4096 14 -> 16 us).
int gemm_plain_tile_rows(int K) { return K >= 128 * BK ? 128 : 64; }

hipError_t launch_gemm_plain(const GemmArgs& a, int ksplit, hipStream_t st) {
  if (gemm_plain_tile_rows(a.K_tail) == 128)
    return launch_cfg<4, false, 128, 128, 2, 4, false, false>(a, ksplit, st);
  return launch_cfg<4, false, 64, 128, 2, 4, false, false>(a, ksplit, st);
}

}  // namespace qalora
