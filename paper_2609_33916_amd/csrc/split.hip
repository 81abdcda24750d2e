// Launches of the kernels for small grids (split.hpp).
#include "launch.hpp"
#include "split.hpp"

namespace attn {

template <typename T, int D, bool CAUSAL> void launch_fwd_split(FwdArgs a, int heads, hipStream_t st) {
  set_grid(a, heads, kSplitRows, 2);
  hipLaunchKernelGGL((fwd_split_kernel<T, D, CAUSAL>), dim3(a.nblocks), dim3(256), 0, st, a);
}
template <typename T, int D, bool CAUSAL, bool AQ> void launch_dkdv_split(BwdArgs a, int heads, hipStream_t st) {
  set_grid(a, heads, kSplitRows, 2);
  hipLaunchKernelGGL((dkdv_split_kernel<T, D, CAUSAL, AQ>), dim3(a.nblocks), dim3(256), 0, st, a);
}
template <typename T, int D, bool CAUSAL> void launch_dq_split(BwdArgs a, int heads, hipStream_t st) {
  set_grid(a, heads, kSplitRows, 2);
  hipLaunchKernelGGL((dq_split_kernel<T, D, CAUSAL>), dim3(a.nblocks), dim3(256), 0, st, a);
}

template <typename T, int D, bool CAUSAL> void launch_bwd_split(BwdArgs a, int heads, hipStream_t st) {
  set_grid(a, heads, kSplitRows, 2);
  hipLaunchKernelGGL((bwd_split_kernel<T, D, CAUSAL>), dim3(2 * a.nblocks), dim3(256), 0, st, a);
}

#define ATTN_SPLIT_INST(T, D, C)                                    \
  template void launch_fwd_split<T, D, C>(FwdArgs, int, hipStream_t);  \
  template void launch_dkdv_split<T, D, C, false>(BwdArgs, int, hipStream_t); \
  template void launch_dq_split<T, D, C>(BwdArgs, int, hipStream_t);   \
  template void launch_bwd_split<T, D, C>(BwdArgs, int, hipStream_t);
#define ATTN_SPLIT_INST_D(T, D) ATTN_SPLIT_INST(T, D, false) ATTN_SPLIT_INST(T, D, true)

ATTN_SPLIT_INST_D(bf16, 32)
ATTN_SPLIT_INST_D(bf16, 64)
ATTN_SPLIT_INST_D(bf16, 128)
ATTN_SPLIT_INST_D(float, 32)
ATTN_SPLIT_INST_D(float, 64)
ATTN_SPLIT_INST_D(float, 128)

#define ATTN_SPLIT_INST_AQ(D)                                                  \
  template void launch_dkdv_split<bf16, D, false, true>(BwdArgs, int, hipStream_t); \
  template void launch_dkdv_split<bf16, D, true, true>(BwdArgs, int, hipStream_t);
ATTN_SPLIT_INST_AQ(32)
ATTN_SPLIT_INST_AQ(64)
ATTN_SPLIT_INST_AQ(128)

#undef ATTN_SPLIT_INST_AQ
#undef ATTN_SPLIT_INST_D
#undef ATTN_SPLIT_INST

}  // namespace attn
