// Spinor streaming whole-step kernel, complex128 with reservoirs.
#include "stream_spinor_launch.h"

namespace phx {
template hipError_t launch_spinor_part<double, 1, true, false, false>(bool, const StepArgs<double>&, hipStream_t);
}  // namespace phx
