// Launch of the streaming whole-step kernel (stream_step.h) for one precision, column count
// and set of terms; the units that instantiate it compile in parallel.
#pragma once

#include "runtime.h"
#include "stream_step.h"

namespace phx {

// IMAG (imaginary time): the wave of tile t writes the FP64 norm partial of its cells to
// a.imag_partials[t], reduced over the lanes in a fixed butterfly order.
template <typename R, int W, bool RES, bool HASV, bool GHOSTS, bool YZERO, bool CHECK, bool IMAG, bool DRIVE, bool NOISE,
          int WPE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPE)))
void rk4_stream_step_kernel(const StepArgs<R> a)
{
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const int band = t / a.tiles_x, strip = t - band * a.tiles_x;
    R sc = R(1);
    if constexpr (IMAG) sc = imag_scale(a);
    const uint64_t nstep = NOISE ? *a.noise_step + (uint64_t)a.noise_offset : 0u;
    stream_band_step<R, W, RES, HASV, GHOSTS, YZERO, CHECK, IMAG, DRIVE, NOISE>(
        a, strip, band, a.band_rows, (band & 1) ? -1 : 1, sc, nstep,
        [&](bool bad, double nrm) __attribute__((always_inline)) {
            if (bad) a.flag[0] = 1u;  // benign race: every writer stores 1
            if constexpr (IMAG) {
#pragma unroll
                for (int m = 32; m >= 1; m >>= 1) nrm += __shfl_xor(nrm, m, 64);
                if (threadIdx.x == 0) a.imag_partials[t] = nrm;
            }
        });
}

template <typename R, int W, bool RES, bool HASV, bool GHOSTS, bool YZERO, bool IMAG, bool DRIVE, bool NOISE>
static void launch_step_walk_t(const StepArgs<R>& a, hipStream_t s)
{
    constexpr int WPE = step_waves_per_simd(W, sizeof(R) == 8, RES, DRIVE);
    if (a.check)
        rk4_stream_step_kernel<R, W, RES, HASV, GHOSTS, YZERO, true, IMAG, DRIVE, NOISE, WPE><<<a.tiles, 64, 0, s>>>(a);
    else
        rk4_stream_step_kernel<R, W, RES, HASV, GHOSTS, YZERO, false, IMAG, DRIVE, NOISE, WPE><<<a.tiles, 64, 0, s>>>(a);
}

template <typename R, int W, bool RES, bool IMAG, bool DRIVE, bool NOISE>
static hipError_t launch_step_walk_v(bool has_v, const StepArgs<R>& a, hipStream_t s)
{
#define PHX_SW(HV) \
    if (has_v == HV) { \
        if (a.bcy == PHX_BC_ZERO) \
            launch_step_walk_t<R, W, RES, HV, true, true, IMAG, DRIVE, NOISE>(a, s); \
        else if (a.bcx == PHX_BC_ZERO) \
            launch_step_walk_t<R, W, RES, HV, true, false, IMAG, DRIVE, NOISE>(a, s); \
        else \
            launch_step_walk_t<R, W, RES, HV, false, false, IMAG, DRIVE, NOISE>(a, s); \
    }
    PHX_SW(false)
    PHX_SW(true)
#undef PHX_SW
    return hipGetLastError();
}

// the undriven walk: plain steps, imaginary time (no reservoir), increments drawn in the
// step (two columns per lane)
template <typename R, int W>
hipError_t launch_step_walk(bool reservoir, bool has_v, const StepArgs<R>& a, hipStream_t s)
{
    if (a.imag_partials)
        return reservoir ? hipErrorInvalidValue : launch_step_walk_v<R, W, false, true, false, false>(has_v, a, s);
    if constexpr (W == 2) {
        if (a.noise_step)
            return reservoir ? launch_step_walk_v<R, W, true, false, false, true>(has_v, a, s)
                             : launch_step_walk_v<R, W, false, false, false, true>(has_v, a, s);
    }
    return reservoir ? launch_step_walk_v<R, W, true, false, false, false>(has_v, a, s)
                     : launch_step_walk_v<R, W, false, false, false, false>(has_v, a, s);
}

// the coherent drive (one column per lane)
template <typename R>
hipError_t launch_step_walk_drive(bool reservoir, bool has_v, const StepArgs<R>& a, hipStream_t s)
{
    return reservoir ? launch_step_walk_v<R, 1, true, false, true, false>(has_v, a, s)
                     : launch_step_walk_v<R, 1, false, false, true, false>(has_v, a, s);
}

}  // namespace phx
