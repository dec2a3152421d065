// Whole-attempt Dormand-Prince kernel, float, two components.
#include "dp_walk_launch.h"

namespace phx {
template hipError_t launch_dp_walk<float, 2>(bool, const DpWalkArgs<float>&, hipStream_t);
}  // namespace phx
