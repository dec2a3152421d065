// Spinor streaming whole-step kernel, complex128 with the coherent drive.
#include "stream_spinor_launch.h"

namespace phx {
template hipError_t launch_spinor_part<double, 1, false, false, true>(bool, const StepArgs<double>&, hipStream_t);
}  // namespace phx
