// Two-step form of the batched stepper, complex128.
#include "batch_pair.h"

namespace phx {
template hipError_t launch_batch_pair_forms<double, 1>(const BatchForm&, int, int, const BatchInst<double>*, int,
                                                      const BatchState<double>&, bool, hipStream_t);
}  // namespace phx
