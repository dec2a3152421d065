// Spinor streaming whole-step kernel, complex64 in imaginary time.
#include "stream_spinor_launch.h"

namespace phx {
template hipError_t launch_spinor_part<float, 1, false, true, false>(bool, const StepArgs<float>&, hipStream_t);
}  // namespace phx
