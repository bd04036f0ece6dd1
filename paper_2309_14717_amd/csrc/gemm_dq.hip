// Launch rules of the dequantising product (gemm_dq_impl.hpp) and the sum over the slices of a split K range.
#include "gemm_dq_impl.hpp"
#include "split_sum.hpp"

namespace qalora {

// (gemm_dq_192.hip)
hipError_t launch_192(int bits, bool bwd, const GemmArgs& a, int ks, hipStream_t st, hipEvent_t e0, hipEvent_t e1);

template <int NBITS, bool BWD>
static hipError_t launch_dir(const GemmArgs& a, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const int ks = a.ksplit > 1 ? a.ksplit : 1;
  if (a.a_main_padded_rows >= round_up(a.M, 256) && gemm_fast_shape(a.K_main, a.group)) {
    if (a.tile_rows == 256) return launch_cfg<NBITS, BWD, 256, 256, 2, 4, true>(a, ks, st, e0, e1);
    if (a.tile_rows == 192) return launch_192(NBITS, BWD, a, ks, st, e0, e1);
    if (a.tile_rows == 128) return launch_cfg<NBITS, BWD, 128, 256, 2, 4, true>(a, ks, st, e0, e1);
    return launch_cfg<NBITS, BWD, 64, 256, 1, 8, true>(a, ks, st, e0, e1);
  }
  if (a.tile_rows > 64) return launch_cfg<NBITS, BWD, 128, 256, 2, 4, false>(a, ks, st, e0, e1);
  return launch_cfg<NBITS, BWD, 64, 256, 1, 8, false>(a, ks, st, e0, e1);
}

// out = sum over the K slices of the partial products, slice order, converted on the way out
__global__ __launch_bounds__(256) void split_reduce_kernel(const SplitSum s) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;  // group of 4 elements
  if (i < s.n4) split_sum_one(s, i);
}

ProfileHook g_profile_hook[2] = {{nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr}};

static hipError_t launch_bits(int bits, bool bwd, const GemmArgs& a, hipStream_t st, hipEvent_t e0,
                              hipEvent_t e1) {
  if (bits == 4) return bwd ? launch_dir<4, true>(a, st, e0, e1) : launch_dir<4, false>(a, st, e0, e1);
  if (bits == 3) return bwd ? launch_dir<3, true>(a, st, e0, e1) : launch_dir<3, false>(a, st, e0, e1);
  return bwd ? launch_dir<2, true>(a, st, e0, e1) : launch_dir<2, false>(a, st, e0, e1);
}

hipError_t launch_gemm_dq(int bits, bool bwd, const GemmArgs& args, hipStream_t st, SplitSum* sum) {
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
  // (the product alone where the caller sums)
  const bool ride = !split && hook.start && hook.stop;
  if (hook.start && !ride) (void)hipEventRecord(hook.start, st);
  hipError_t e = launch_bits(bits, bwd, a, st, ride ? hook.start : nullptr, ride ? hook.stop : nullptr);
  if (e == hipSuccess && split) {
    const SplitSum todo{a.partial, a.ksplit, (size_t)a.M * a.N / 4, args.out, args.out_bf16};  // N is a multiple of 8
    if (sum) {
      *sum = todo;
    } else {
      split_reduce_kernel<<<(unsigned)((todo.n4 + 255) / 256), 256, 0, st>>>(todo);
      e = hipGetLastError();
    }
  }
  if (hook.stop && !ride) (void)hipEventRecord(hook.stop, st);
  return e;
}

}  // namespace qalora
