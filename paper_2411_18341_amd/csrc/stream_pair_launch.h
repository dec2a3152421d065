// Launch of the two-step streaming kernel (stream_pair.h) for one precision and column
// count; each is instantiated in a unit of its own.
#pragma once

#include "runtime.h"
#include "stream_pair.h"

namespace phx {

template <typename R, int W, bool RES, bool HASV, bool GHOSTS, bool YZERO, bool DRIVE>
static void launch_pair_t(const StepArgs<R>& a, hipStream_t s)
{
    constexpr int WPE = pair_waves_per_simd(W * (int)sizeof(R) / 4, RES, HASV, GHOSTS, DRIVE);
    if (a.check)
        rk4_stream_pair_kernel<R, W, RES, HASV, GHOSTS, YZERO, WPE, true, DRIVE><<<a.tiles, 64, 0, s>>>(a);
    else
        rk4_stream_pair_kernel<R, W, RES, HASV, GHOSTS, YZERO, WPE, false, DRIVE><<<a.tiles, 64, 0, s>>>(a);
}

template <typename R, int W, bool RES, bool HASV, bool DRIVE = false>
static hipError_t launch_pair_v(const StepArgs<R>& a, hipStream_t s)
{
    if (a.bcy == PHX_BC_PERIODIC && a.bcx == PHX_BC_PERIODIC) {
        launch_pair_t<R, W, RES, HASV, false, false, DRIVE>(a, s);
    } else if constexpr (pair_pays(W * (int)sizeof(R) / 4, RES, HASV, true)) {
        if (a.bcy == PHX_BC_ZERO)
            launch_pair_t<R, W, RES, HASV, true, true, DRIVE>(a, s);
        else
            launch_pair_t<R, W, RES, HASV, true, false, DRIVE>(a, s);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename R, int W>
hipError_t launch_stream_pair(bool reservoir, bool has_v, const StepArgs<R>& a, hipStream_t s)
{
    if (reservoir) return has_v ? launch_pair_v<R, W, true, true>(a, s) : launch_pair_v<R, W, true, false>(a, s);
    return has_v ? launch_pair_v<R, W, false, true>(a, s) : launch_pair_v<R, W, false, false>(a, s);
}

// with the coherent drive (one column per lane; complex128 without a potential)
template <typename R>
hipError_t launch_stream_pair_drive(bool reservoir, bool has_v, const StepArgs<R>& a, hipStream_t s)
{
    if constexpr (sizeof(R) == 4) {
        if (has_v) return reservoir ? launch_pair_v<R, 1, true, true, true>(a, s) : launch_pair_v<R, 1, false, true, true>(a, s);
    }
    if (has_v) return hipErrorInvalidValue;
    return reservoir ? launch_pair_v<R, 1, true, false, true>(a, s) : launch_pair_v<R, 1, false, false, true>(a, s);
}

}  // namespace phx
