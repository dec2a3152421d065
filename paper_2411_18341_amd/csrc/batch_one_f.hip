// One-step batched walk, one column per lane, float.
#include "batch_walk.h"

namespace phx {
template hipError_t launch_batch_step_forms<float, 1, false>(const BatchForm&, int, int, const BatchInst<float>*, int,
                                                            const BatchState<float>&, uint64_t, bool, hipStream_t);
}  // namespace phx
