// Two-step wide streaming RK4 kernel (complex64, one component; stream_pair.h).
#include "runtime.h"
#include "stream_pair.h"

namespace phx {

template <bool RES, bool HASV, bool GHOSTS, bool YZERO>
static void launch_pair_t(const StepArgs<float>& a, hipStream_t s)
{
    constexpr int WPE = pair_waves_per_simd(RES, HASV, GHOSTS);
    if (a.check)
        rk4_stream_pair_kernel<RES, HASV, GHOSTS, YZERO, WPE, true><<<a.tiles, 64, 0, s>>>(a);
    else
        rk4_stream_pair_kernel<RES, HASV, GHOSTS, YZERO, WPE, false><<<a.tiles, 64, 0, s>>>(a);
}

template <bool RES, bool HASV>
static hipError_t launch_pair_v(const StepArgs<float>& a, hipStream_t s)
{
    if (a.bcy == PHX_BC_ZERO)
        launch_pair_t<RES, HASV, true, true>(a, s);
    else if (a.bcx == PHX_BC_ZERO)
        launch_pair_t<RES, HASV, true, false>(a, s);
    else
        launch_pair_t<RES, HASV, false, false>(a, s);
    return hipGetLastError();
}

hipError_t launch_stream_pair(bool reservoir, bool has_v, const StepArgs<float>& a, hipStream_t s)
{
    if (reservoir) return has_v ? launch_pair_v<true, true>(a, s) : launch_pair_v<true, false>(a, s);
    return has_v ? launch_pair_v<false, true>(a, s) : launch_pair_v<false, false>(a, s);
}

}  // namespace phx
