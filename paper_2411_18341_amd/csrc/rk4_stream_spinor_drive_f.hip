// Spinor streaming whole-step kernel, complex64 with the coherent drive.
#include "stream_spinor_launch.h"

namespace phx {
template hipError_t launch_spinor_part<float, 1, false, false, true>(bool, const StepArgs<float>&, hipStream_t);
}  // namespace phx
