// Launch rules of the dequantising product (gemm_dq_impl.hpp), the sum over the slices of a split K range,
// and the plain product of the adapter gradients.
#include "gemm_dq_impl.hpp"

namespace qalora {

// 192-row tiles instead of 256-row ones.  A K step of theirs takes 0.8 of a 256-row one (the producer's share
// does not shrink), so they pay where they save rows of padding or a ragged last round of blocks:
// 2-bit 5120 x 13824, us per call with 256 / 192 rows: 192 tokens 61.5 / 55.6, 320 90.7 / 78, 700 118 / 112,
// 1531 248 / 219; 4096 x 11008 with 3 bits at 2048 tokens 218 / 202; level where both need the same
// number of rounds times rows.  The split of K stays what gemm_dq_ksplit plans for 256-row tiles (tile and split
// are not searched together), and every element is summed in the same order by the same instructions:
// the results are the same bits.
static bool prefer_192(const GemmArgs& a, int ks) {
  auto cost = [&](int bm, double step) {
    const long blocks = (long)ceil_div(a.M, bm) * ceil_div(a.N, 256) * ks;
    return (double)((blocks + 255) / 256) * step;
  };
  return cost(192, 0.8) < cost(256, 1.0);
}
// (gemm_dq_192.hip)
hipError_t launch_192(int bits, bool bwd, const GemmArgs& a, int ks, hipStream_t st, hipEvent_t e0, hipEvent_t e1);

template <int NBITS, bool BWD>
static hipError_t launch_dir(const GemmArgs& a, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const int ks = a.ksplit > 1 ? a.ksplit : 1;
  const bool fast = a.a_main_padded_rows >= round_up(a.M, 256) && a.K_main % BK == 0 &&
                    (BK % a.group == 0 || a.group % BK == 0);
  if (a.M > 128) {
    if (fast && prefer_192(a, ks)) return launch_192(NBITS, BWD, a, ks, st, e0, e1);
    if (fast) return launch_cfg<NBITS, BWD, 256, 256, 2, 4, true, true>(a, ks, st, e0, e1);
    return launch_cfg<NBITS, BWD, 128, 256, 2, 4, true, false>(a, ks, st, e0, e1);
  }
  if (a.M > 64) {
    if (fast) return launch_cfg<NBITS, BWD, 128, 256, 2, 4, true, true>(a, ks, st, e0, e1);
    return launch_cfg<NBITS, BWD, 128, 256, 2, 4, true, false>(a, ks, st, e0, e1);
  }
  if (fast) return launch_cfg<NBITS, BWD, 64, 256, 1, 8, true, true>(a, ks, st, e0, e1);
  return launch_cfg<NBITS, BWD, 64, 256, 1, 8, true, false>(a, ks, st, e0, e1);
}

// K splits of the dequantising product.  One block runs per compute unit, so a launch takes
// rounds(tiles x splits) x (steps per block + a fixed cost per block); splitting K pays when it
// fills compute units that a short or ragged last round leaves idle (few tokens; 160 tiles on
// 256 units) by more than the fp32 partial sums cost: `splits` copies of the output written
// here and read again by the sum, priced at 4 TB/s against the ~2 us of a 256-row K step.
// At least eight K steps per slice.
int gemm_dq_ksplit(int M, int N, int K_main) {
  constexpr double kBlockSteps = 7;  // prologue + epilogue of a block, in K steps
  const int bm = M > 128 ? 256 : (M > 64 ? 128 : 64);
  const int kUnits = bm == 64 ? 512 : 256;  // resident blocks: one per compute unit, two of the 64-row tile
  const long tiles = (long)ceil_div(M, bm) * ceil_div(N, 256);
  const int nk = ceil_div(K_main, BK);
  const double step_us = 2.0 * bm / 256;
  auto cost = [&](int ks) {
    const long rounds = (tiles * ks + kUnits - 1) / kUnits;
    const double sum_us = ks > 1 ? (double)M * N * (8.0 * ks + 2.0) / 4e6 : 0.0;
    return rounds * (ceil_div(nk, ks) + kBlockSteps) + sum_us / step_us;
  };
  int best = 1;
  double best_cost = cost(1);
  for (int ks = 2; ks <= 16 && nk / ks >= 8; ++ks) {
    const double c = cost(ks);
    if (c < best_cost) {
      best_cost = c;
      best = ks;
    }
  }
  return best;
}

// out = sum over the K slices of the partial products, slice order, converted on the way out
__global__ __launch_bounds__(256) void split_reduce_kernel(const float* __restrict__ part,
                                                           int nparts, size_t n4, void* out,
                                                           int out_bf16) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;  // group of 4 elements
  if (i >= n4) return;
  f32x4 v = reinterpret_cast<const f32x4*>(part)[i];
  for (int z = 1; z < nparts; ++z) v += reinterpret_cast<const f32x4*>(part)[(size_t)z * n4 + i];
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
