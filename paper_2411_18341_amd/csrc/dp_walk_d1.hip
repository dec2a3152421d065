// Whole-attempt Dormand-Prince kernel, double, one component.
#include "dp_walk_launch.h"

namespace phx {
template hipError_t launch_dp_walk<double, 1>(bool, const DpWalkArgs<double>&, hipStream_t);
}  // namespace phx
