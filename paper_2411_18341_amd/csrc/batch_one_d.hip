// One-step batched walk, one column per lane, double.
#include "batch_walk.h"

namespace phx {
template hipError_t launch_batch_step_forms<double, 1, false>(const BatchForm&, int, int, const BatchInst<double>*, int,
                                                            const BatchState<double>&, uint64_t, bool, hipStream_t);
}  // namespace phx
