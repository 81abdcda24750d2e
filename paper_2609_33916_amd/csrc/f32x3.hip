// Launches of the float32 kernels on the bfloat16 matrix cores (f32x3.hpp):
// 64-row tiles (32 at d = 128, and for the four-wave dK/dV at d = 64, which has
// no registers for more; 128 for eight waves at d = 32, a whole chunk for each
// thread).
#include "launch.hpp"
#include "f32x3.hpp"

namespace attn {

template <int D, bool CAUSAL> void launch_fwd_x3(FwdArgs a, int heads, hipStream_t st) {
  set_grid(a, heads, 128, 2);
  if constexpr (D != 128) {
    if (x3_eight_waves(D, CAUSAL, heads, a.n)) {
      hipLaunchKernelGGL((fwd_x3_kernel<D, CAUSAL, 2, D == 32 ? 128 : 64>), dim3(a.nblocks), dim3(512), 0, st, a);
      return;
    }
  }
  hipLaunchKernelGGL((fwd_x3_kernel<D, CAUSAL, 1, D == 128 ? 32 : 64>), dim3(a.nblocks), dim3(256), 0, st, a);
}
template <int D, bool CAUSAL> void launch_dkdv_x3(BwdArgs a, int heads, hipStream_t st) {
  set_grid(a, heads, 128, D == 128 ? 1 : 2);
  if constexpr (D != 128) {
    if (x3_eight_waves(D, CAUSAL, heads, a.n)) {
      hipLaunchKernelGGL((dkdv_x3_kernel<D, CAUSAL, 2, D == 32 ? 128 : 64>), dim3(a.nblocks), dim3(512), 0, st, a);
      return;
    }
  }
  hipLaunchKernelGGL((dkdv_x3_kernel<D, CAUSAL, 1, D == 32 ? 64 : 32>), dim3(a.nblocks), dim3(256), 0, st, a);
}
template <int D, bool CAUSAL> void launch_dq_x3(BwdArgs a, int heads, hipStream_t st) {
  set_grid(a, heads, 128, D == 128 ? 1 : 2);
  if constexpr (D != 128) {
    if (x3_eight_waves(D, CAUSAL, heads, a.n)) {
      hipLaunchKernelGGL((dq_x3_kernel<D, CAUSAL, 2, D == 32 ? 128 : 64>), dim3(a.nblocks), dim3(512), 0, st, a);
      return;
    }
  }
  hipLaunchKernelGGL((dq_x3_kernel<D, CAUSAL, 1, D == 128 ? 32 : 64>), dim3(a.nblocks), dim3(256), 0, st, a);
}

#define ATTN_X3_INST(D, C)                                   \
  template void launch_fwd_x3<D, C>(FwdArgs, int, hipStream_t);  \
  template void launch_dkdv_x3<D, C>(BwdArgs, int, hipStream_t); \
  template void launch_dq_x3<D, C>(BwdArgs, int, hipStream_t);
ATTN_X3_INST(32, false)
ATTN_X3_INST(32, true)
ATTN_X3_INST(64, false)
ATTN_X3_INST(64, true)
ATTN_X3_INST(128, false)
ATTN_X3_INST(128, true)
#undef ATTN_X3_INST

}  // namespace attn
