// Spinor streaming whole-step kernel, complex128 in imaginary time.
#include "stream_spinor_launch.h"

namespace phx {
template hipError_t launch_spinor_part<double, 1, false, true, false>(bool, const StepArgs<double>&, hipStream_t);
}  // namespace phx
