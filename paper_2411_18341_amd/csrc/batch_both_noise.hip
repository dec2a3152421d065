// One-step batched walk, instances of both column counts; the increments of those with two
// columns per lane are drawn in the step.
#include "batch_walk.h"

namespace phx {
template hipError_t launch_batch_step_forms<float, 3, true>(const BatchForm&, int, int, const BatchInst<float>*, int,
                                                            const BatchState<float>&, uint64_t, bool, hipStream_t);
}  // namespace phx
