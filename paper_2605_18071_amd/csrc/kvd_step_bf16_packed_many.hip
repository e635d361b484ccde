#include "kvd_step_launch.h"

template void kvd::launch_step<true, kvd::kLayoutPacked, true>(int, const StepArgs&, int, hipStream_t);
