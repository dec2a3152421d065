// Two-step form of the batched stepper, complex64, two columns per lane.
#include "batch_pair.h"

namespace phx {
template hipError_t launch_batch_pair_w<float, 2>(bool, bool, bool, bool, int, const BatchInst<float>*, int, const void*,
                                                 const void*, void*, void*, const void*, const void*, unsigned int*,
                                                 bool, hipStream_t);
}  // namespace phx
