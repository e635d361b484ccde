#include "kvd_step_launch.h"

template void kvd::launch_step<true, kvd::kLayoutTiles, true>(int, const StepArgs&, int, hipStream_t);
