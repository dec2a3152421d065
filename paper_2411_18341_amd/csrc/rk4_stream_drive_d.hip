// Streaming RK4 kernels, one and two steps per launch, with the coherent drive of Eq.
// (PULSE_psi), double: the drive profile rides in the input ring, the phasors of the stage
// times (written from the device step index) join every stage's derivative.
#include "stream_pair_launch.h"
#include "stream_step_launch.h"

namespace phx {
template hipError_t launch_step_walk_drive<double>(bool, bool, const StepArgs<double>&, hipStream_t);
template hipError_t launch_stream_pair_drive<double>(bool, bool, const StepArgs<double>&, hipStream_t);
}  // namespace phx
