#include "kvd_step_launch.h"

template void kvd::launch_step<false, kvd::kLayoutPacked, false>(int, const StepArgs&, int, hipStream_t);
