// Streaming whole-step RK4 kernel, complex64, two columns per lane (also with the increments drawn in the step).
#include "stream_step_launch.h"

namespace phx {
template hipError_t launch_step_walk<float, 2>(bool, bool, const StepArgs<float>&, hipStream_t);
}  // namespace phx
