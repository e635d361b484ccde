#include "kvd_step_launch.h"

template void kvd::launch_step<false, kvd::kLayoutNatural, false>(int, const StepArgs&, int, hipStream_t);
