// Whole-attempt Dormand-Prince kernel, double, two components.
#include "dp_walk_launch.h"

namespace phx {
template hipError_t launch_dp_walk<double, 2>(bool, const DpWalkArgs<double>&, hipStream_t);
}  // namespace phx
