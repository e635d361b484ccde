#include "kvd_step_launch.h"

template void kvd::launch_step<true, true, true>(int, int, const StepArgs&, int, hipStream_t);
