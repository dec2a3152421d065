// Two-step form of the batched stepper, complex64, instances of both column counts.
#include "batch_pair.h"

namespace phx {
template hipError_t launch_batch_pair_forms<float, 3>(const BatchForm&, int, int, const BatchInst<float>*, int,
                                                      const BatchState<float>&, bool, hipStream_t);
}  // namespace phx
