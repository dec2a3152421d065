// Two-step streaming RK4 kernel, complex64, two columns per lane.
#include "stream_pair_launch.h"

namespace phx {
template hipError_t launch_stream_pair<float, 2>(bool, bool, const StepArgs<float>&, hipStream_t);
}  // namespace phx
