// Streaming whole-step RK4 kernel, complex128.
#include "stream_step_launch.h"

namespace phx {
template hipError_t launch_step_walk<double, 1>(bool, bool, const StepArgs<double>&, hipStream_t);
}  // namespace phx
