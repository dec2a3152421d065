// Two-step streaming RK4 kernel, complex128.
#include "stream_pair_launch.h"

namespace phx {
template hipError_t launch_stream_pair<double, 1>(bool, bool, const StepArgs<double>&, hipStream_t);
}  // namespace phx
