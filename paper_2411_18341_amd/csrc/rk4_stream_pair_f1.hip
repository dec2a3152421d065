// Two-step streaming RK4 kernel, complex64, one column per lane.
#include "stream_pair_launch.h"

namespace phx {
template hipError_t launch_stream_pair<float, 1>(bool, bool, const StepArgs<float>&, hipStream_t);
}  // namespace phx
