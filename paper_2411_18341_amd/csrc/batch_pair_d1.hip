// Two-step form of the batched stepper, complex128.
#include "batch_pair.h"

namespace phx {
template hipError_t launch_batch_pair_w<double, 1>(bool, bool, bool, bool, int, const BatchInst<double>*, int, const void*,
                                                 const void*, void*, void*, const void*, const void*, unsigned int*,
                                                 bool, hipStream_t);
}  // namespace phx
