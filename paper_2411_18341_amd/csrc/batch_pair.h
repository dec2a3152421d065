// Two-step form of the batched stepper (the walk of stream_pair.h): a work item is one band
// of one strip of one instance, one single-wave workgroup per item (consecutive items on one
// XCD).  The instances with two columns per lane form one list, those with one another; a
// batch that has both runs them in one launch (FORMS = 3), the longer items of the first
// list before the others, with the registers of the first.  (As two launches on two streams,
// forked and joined by events, a pair of steps of 16 grids around 128^2 took 56 us, now 28; 256
// grids of 128^2 to 1024^2, four steps, 1237 -> 1218.)
#pragma once

#include "batch_inst.h"
#include "stream_pair.h"

namespace phx {

template <typename R, int W, bool RES, bool HASV, bool GHOSTS, bool YZERO, bool CHECK>
__device__ __forceinline__ void batch_pair_item(const BatchInst<R>* __restrict__ inst, int count,
                                                const BatchState<R>& b, int t)
{
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (inst[mid].p_tile0[W - 1] <= t) lo = mid; else hi = mid - 1;
    }
    const BatchInst<R>& I = inst[lo];
    const int lt = t - I.p_tile0[W - 1];
    const int band = lt / I.p_strips, strip = lt - band * I.p_strips;
    StepArgs<R> a{};
    a.nx = I.nx;
    a.ny = I.ny;
    a.bcx = I.bcx;
    a.bcy = I.bcy;
    a.c = I.c;
    a.half_dt = I.half_dt;
    a.dt = I.dt;
    a.dt6 = I.dt6;
    a.psi_in = b.psi_in + I.offset;
    a.n_in = RES ? b.n_in + I.offset : nullptr;
    a.psi_out = b.psi_out + I.offset;
    a.n_out = RES ? b.n_out + I.offset : nullptr;
    a.V = HASV ? b.V + I.offset : nullptr;
    a.P = RES ? b.P + I.offset : nullptr;
    stream_band_pair<R, W, RES, HASV, GHOSTS, YZERO, CHECK, false>(a, strip, band, I.p_band, (band & 1) ? -1 : 1,
                                                           [&](bool bad) __attribute__((always_inline)) {
                                                               if (bad) b.flag[0] = 1u;  // benign race
                                                           });
}

// FORMS: column counts in the launch (1, 2, or 3 for both); total2: items with two columns
template <typename R, int FORMS, bool RES, bool HASV, bool GHOSTS, bool YZERO, bool CHECK, int WPE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPE)))
void batch_stream_pair_kernel(const BatchInst<R>* __restrict__ inst, int count, const BatchState<R> b, int total2)
{
    const int v = blockIdx.x;
    if constexpr (FORMS != 1) {
        if (FORMS == 2 || v < total2) {
            batch_pair_item<R, 2, RES, HASV, GHOSTS, YZERO, CHECK>(inst, count, b, xcd_tile(v, total2));
            return;
        }
    }
    if constexpr (FORMS != 2)
        batch_pair_item<R, 1, RES, HASV, GHOSTS, YZERO, CHECK>(inst, count, b,
                                                              xcd_tile(v - total2, gridDim.x - total2));
}

template <typename R, int FORMS, bool RES, bool HASV, bool GHOSTS, bool YZERO>
static hipError_t launch_batch_pair_t(int total1, int total2, const BatchInst<R>* inst, int count, const BatchState<R>& b,
                                bool check, hipStream_t s)
{
    constexpr int W = FORMS == 1 ? 1 : 2;
    constexpr int words = W * (int)sizeof(R) / 4;
    constexpr int WPE = pair_waves_per_simd(words, RES, HASV, GHOSTS, false);
    if constexpr (batch_pair_built(words, sizeof(R) == 8, RES, HASV, GHOSTS, YZERO)) {
        if (check)
            batch_stream_pair_kernel<R, FORMS, RES, HASV, GHOSTS, YZERO, true, WPE>
                <<<total1 + total2, 64, 0, s>>>(inst, count, b, total2);
        else
            batch_stream_pair_kernel<R, FORMS, RES, HASV, GHOSTS, YZERO, false, WPE>
                <<<total1 + total2, 64, 0, s>>>(inst, count, b, total2);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

template <typename R, int FORMS>
hipError_t launch_batch_pair_forms(const BatchForm& f, int total1, int total2, const BatchInst<R>* inst, int count,
                                   const BatchState<R>& b, bool check, hipStream_t s)
{
#define PHX_BP(RS, HV) \
    if (f.res == RS && f.hasv == HV) { \
        if (f.yzero) \
            return launch_batch_pair_t<R, FORMS, RS, HV, true, true>(total1, total2, inst, count, b, check, s); \
        else if (f.ghosts) \
            return launch_batch_pair_t<R, FORMS, RS, HV, true, false>(total1, total2, inst, count, b, check, s); \
        else \
            return launch_batch_pair_t<R, FORMS, RS, HV, false, false>(total1, total2, inst, count, b, check, s); \
    }
    PHX_BP(true, true)
    PHX_BP(true, false)
    PHX_BP(false, true)
    PHX_BP(false, false)
#undef PHX_BP
    return hipErrorInvalidValue;
}

}  // namespace phx
