// Launch of the whole-attempt Dormand-Prince kernel (dp_walk.h) for one precision and
// component count; each pair is instantiated in a unit of its own (they compile in
// parallel).
#pragma once

#include "dp_walk.h"
#include "runtime.h"

namespace phx {

template <typename R, int COMPS, bool RES, bool HASV, bool SKIP>
static void launch_dp_walk_s(bool ghosts, const DpWalkArgs<R>& a, hipStream_t s)
{
    constexpr int WPE = dp_waves_per_simd(sizeof(R) == 4, COMPS, RES, HASV, SKIP);
    if (ghosts)
        dp_stream_kernel<R, COMPS, RES, HASV, true, SKIP, WPE><<<a.tiles, 64, 0, s>>>(a);
    else
        dp_stream_kernel<R, COMPS, RES, HASV, false, SKIP, WPE><<<a.tiles, 64, 0, s>>>(a);
}

// Leaving out the stages that no output needs saves 56 of the 7 (B + 14) stage rows of a
// walk and costs 5 to 13 % more instructions (copies where the skipped paths join):
// complex64 spinor 158.9 against 173.8 us at 2048^2 (B 41), 524.1 against 512.8 us at
// 4096^2 (B 171); complex128 driven 36.8 against 43.1 us at 513 x 389 (B 5), 161.4
// against 149.7 us at 2048^2 (B 82).
template <typename R, int COMPS, bool RES, bool HASV>
static void launch_dp_walk_t(bool ghosts, const DpWalkArgs<R>& a, hipStream_t s)
{
    if (a.band_rows < kDpSkipRows)
        launch_dp_walk_s<R, COMPS, RES, HASV, true>(ghosts, a, s);
    else
        launch_dp_walk_s<R, COMPS, RES, HASV, false>(ghosts, a, s);
}

template <typename R, int COMPS>
hipError_t launch_dp_walk(bool res, const DpWalkArgs<R>& a, hipStream_t s)
{
    const bool ghosts = a.bcx == PHX_BC_ZERO || a.bcy == PHX_BC_ZERO, hv = a.V != nullptr;
    if constexpr (sizeof(R) == 4 || COMPS == 1) {
        if (res) {
            if (hv)
                launch_dp_walk_t<R, COMPS, true, true>(ghosts, a, s);
            else
                launch_dp_walk_t<R, COMPS, true, false>(ghosts, a, s);
            return hipGetLastError();
        }
    }
    if (res) return hipErrorInvalidValue;
    if (hv)
        launch_dp_walk_t<R, COMPS, false, true>(ghosts, a, s);
    else
        launch_dp_walk_t<R, COMPS, false, false>(ghosts, a, s);
    return hipGetLastError();
}

}  // namespace phx
