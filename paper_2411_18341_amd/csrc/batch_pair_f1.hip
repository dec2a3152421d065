// Two-step form of the batched stepper, complex64, one column per lane.
#include "batch_pair.h"

namespace phx {
template hipError_t launch_batch_pair_w<float, 1>(bool, bool, bool, bool, int, const BatchInst<float>*, int, const void*,
                                                 const void*, void*, void*, const void*, const void*, unsigned int*,
                                                 bool, hipStream_t);
}  // namespace phx
