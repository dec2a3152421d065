// Streaming whole-step RK4 kernel for the two-component (spinor) form
// (stream_spinor.h) and its launch for one precision, column count and set of terms;
// each is instantiated in a unit of its own (they compile in parallel).
#pragma once
#include "runtime.h"
#include "stream_spinor.h"

namespace phx {

// IMAG (imaginary time): the wave of tile t writes the FP64 norm partial of its cells
// (both components) to a.imag_partials[t], reduced over the lanes in a fixed butterfly
// order.
template <typename R, int W, bool RES, bool HASV, bool GHOSTS, bool YZERO, bool IMAG, bool DRIVE, int WPE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPE)))
void rk4_stream_spinor_kernel(const StepArgs<R> a)
{
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const int band = t / a.tiles_x, strip = t - band * a.tiles_x;
    stream_band_spinor<R, W, RES, HASV, GHOSTS, YZERO, IMAG, DRIVE>(
        a, strip, band, a.band_rows, (band & 1) ? -1 : 1, [&](bool bad, double nrm) __attribute__((always_inline)) {
            if (bad) a.flag[0] = 1u;  // benign race
            if constexpr (IMAG) {
#pragma unroll
                for (int m = 32; m >= 1; m >>= 1) nrm += __shfl_xor(nrm, m, 64);
                if (threadIdx.x == 0) a.imag_partials[t] = nrm;
            }
        });
}

template <typename R, int W, bool RES, bool HASV, bool IMAG, bool DRIVE>
static hipError_t launch_spinor_t(const StepArgs<R>& a, hipStream_t s)
{
    constexpr int WPE = spinor_waves_per_simd(sizeof(R) == 4, W, RES, IMAG, DRIVE);
    if (a.bcy == PHX_BC_ZERO)
        rk4_stream_spinor_kernel<R, W, RES, HASV, true, true, IMAG, DRIVE, WPE><<<a.tiles, 64, 0, s>>>(a);
    else if (a.bcx == PHX_BC_ZERO)
        rk4_stream_spinor_kernel<R, W, RES, HASV, true, false, IMAG, DRIVE, WPE><<<a.tiles, 64, 0, s>>>(a);
    else
        rk4_stream_spinor_kernel<R, W, RES, HASV, false, false, IMAG, DRIVE, WPE><<<a.tiles, 64, 0, s>>>(a);
    return hipGetLastError();
}

template <typename R, int W, bool RES, bool IMAG, bool DRIVE>
hipError_t launch_spinor_part(bool has_v, const StepArgs<R>& a, hipStream_t s)
{
    return has_v ? launch_spinor_t<R, W, RES, true, IMAG, DRIVE>(a, s)
                 : launch_spinor_t<R, W, RES, false, IMAG, DRIVE>(a, s);
}

}  // namespace phx
