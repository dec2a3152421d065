// Streaming whole-step RK4 kernel, complex64, one column per lane.
#include "stream_step_launch.h"

namespace phx {
template hipError_t launch_step_walk<float, 1>(bool, bool, const StepArgs<float>&, hipStream_t);
}  // namespace phx
