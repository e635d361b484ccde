// The kernels of the one-launch step, instantiated by source files of one dtype, layout and kind of launch each.
#pragma once
#include "kvd_step_body.h"

namespace kvd {

template <bool BF16, int LAYOUT, bool MANY>
void launch_step(int ipt, const StepArgs& a, int n_blocks, hipStream_t s) {
  dim3 grid(n_blocks), block(kStepThreads);
  if (ipt <= 4) hipLaunchKernelGGL((step_kernel<BF16, kStepThreads, 4, LAYOUT, MANY>), grid, block, 0, s, a);
  else if (ipt <= 8) hipLaunchKernelGGL((step_kernel<BF16, kStepThreads, 8, LAYOUT, MANY>), grid, block, 0, s, a);
  else if (ipt <= 16) hipLaunchKernelGGL((step_kernel<BF16, kStepThreads, 16, LAYOUT, MANY>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((step_kernel<BF16, kStepThreads, 32, LAYOUT, MANY>), grid, block, 0, s, a);
}

}  // namespace kvd
