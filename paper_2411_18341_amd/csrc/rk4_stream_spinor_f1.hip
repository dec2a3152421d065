// Spinor streaming whole-step kernel, complex64, one column per lane.
#include "stream_spinor_launch.h"

namespace phx {
template hipError_t launch_spinor_part<float, 1, false, false, false>(bool, const StepArgs<float>&, hipStream_t);
}  // namespace phx
