// The dequantising product on 192-row tiles (when: gemm_plan.hpp).  A file of its own:
// inside the other's code object a 4096-token step of 4096 x 4096, which does not use these kernels, measured
// 0.6 % slower on the same instructions at other addresses.  (At the edge of what runs differ by; the cause
// was not found.)
#include "gemm_dq_impl.hpp"

namespace qalora {

template <int NBITS>
static hipError_t launch_192_dir(bool bwd, const GemmArgs& a, int ks, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  return bwd ? launch_cfg<NBITS, true, 192, 256, 2, 4, true>(a, ks, st, e0, e1)
             : launch_cfg<NBITS, false, 192, 256, 2, 4, true>(a, ks, st, e0, e1);
}
hipError_t launch_192(int bits, bool bwd, const GemmArgs& a, int ks, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  if (bits == 4) return launch_192_dir<4>(bwd, a, ks, st, e0, e1);
  return bits == 3 ? launch_192_dir<3>(bwd, a, ks, st, e0, e1) : launch_192_dir<2>(bwd, a, ks, st, e0, e1);
}

}  // namespace qalora
