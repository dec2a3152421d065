// Whole-attempt Dormand-Prince kernel, float, one component.
#include "dp_walk_launch.h"

namespace phx {
template hipError_t launch_dp_walk<float, 1>(bool, const DpWalkArgs<float>&, hipStream_t);
}  // namespace phx
