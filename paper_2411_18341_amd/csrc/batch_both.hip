// One-step batched walk, instances of both column counts.
#include "batch_walk.h"

namespace phx {
template hipError_t launch_batch_step_forms<float, 3, false>(const BatchForm&, int, int, const BatchInst<float>*, int,
                                                            const BatchState<float>&, uint64_t, bool, hipStream_t);
}  // namespace phx
