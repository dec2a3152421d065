// One-step streaming form of the batched stepper (the walk of stream_step.h), work items,
// lists and launches as in batch_pair.h.
#pragma once

#include "batch_inst.h"
#include "stream_step.h"

namespace phx {

// NOISE: the increment of step `step` joins the stored cells (two columns per lane)
template <typename R, int W, bool RES, bool HASV, bool GHOSTS, bool YZERO, bool CHECK, bool NOISE>
__device__ __forceinline__ void batch_step_item(const BatchInst<R>* __restrict__ inst, int count,
                                                const BatchState<R>& b, uint64_t step, int t)
{
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (inst[mid].s_tile0[W - 1] <= t) lo = mid; else hi = mid - 1;
    }
    const BatchInst<R>& I = inst[lo];
    const int lt = t - I.s_tile0[W - 1];
    const int band = lt / I.s_strips, strip = lt - band * I.s_strips;
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
    if constexpr (NOISE) {
        a.noise_a = I.noise_a;
        a.noise_b = I.noise_b;
        a.noise_k0 = I.key0;
        a.noise_k1 = I.key1;
    }
    stream_band_step<R, W, RES, HASV, GHOSTS, YZERO, CHECK, false, false, NOISE>(
        a, strip, band, I.s_band, (band & 1) ? -1 : 1, R(1), step, [&](bool bad, double) __attribute__((always_inline)) {
            if (bad) b.flag[0] = 1u;  // benign race: every writer stores 1
        });
}

// FORMS: column counts in the launch (1, 2, or 3 for both); total2: items with two columns
template <typename R, int FORMS, bool RES, bool HASV, bool GHOSTS, bool YZERO, bool CHECK, bool NOISE, int WPE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPE)))
void batch_stream_kernel(const BatchInst<R>* __restrict__ inst, int count, const BatchState<R> b, int total2,
                         uint64_t step)
{
    const int v = blockIdx.x;
    if constexpr (FORMS != 1) {
        if (FORMS == 2 || v < total2) {
            batch_step_item<R, 2, RES, HASV, GHOSTS, YZERO, CHECK, NOISE>(inst, count, b, step, xcd_tile(v, total2));
            return;
        }
    }
    if constexpr (FORMS != 2)
        batch_step_item<R, 1, RES, HASV, GHOSTS, YZERO, CHECK, false>(inst, count, b, step,
                                                                     xcd_tile(v - total2, gridDim.x - total2));
}

template <typename R, int FORMS, bool RES, bool HASV, bool GHOSTS, bool YZERO, bool NOISE>
static void launch_batch_step_t(int total1, int total2, const BatchInst<R>* inst, int count, const BatchState<R>& b,
                                uint64_t step, bool check, hipStream_t s)
{
    constexpr int WPE = step_waves_per_simd(FORMS == 1 ? 1 : 2, sizeof(R) == 8, RES, false);
    if (check)
        batch_stream_kernel<R, FORMS, RES, HASV, GHOSTS, YZERO, true, NOISE, WPE>
            <<<total1 + total2, 64, 0, s>>>(inst, count, b, total2, step);
    else
        batch_stream_kernel<R, FORMS, RES, HASV, GHOSTS, YZERO, false, NOISE, WPE>
            <<<total1 + total2, 64, 0, s>>>(inst, count, b, total2, step);
}

template <typename R, int FORMS, bool NOISE>
hipError_t launch_batch_step_forms(const BatchForm& f, int total1, int total2, const BatchInst<R>* inst, int count,
                                   const BatchState<R>& b, uint64_t step, bool check, hipStream_t s)
{
#define PHX_BS(RS, HV) \
    if (f.res == RS && f.hasv == HV) { \
        if (f.yzero) \
            launch_batch_step_t<R, FORMS, RS, HV, true, true, NOISE>(total1, total2, inst, count, b, step, check, s); \
        else if (f.ghosts) \
            launch_batch_step_t<R, FORMS, RS, HV, true, false, NOISE>(total1, total2, inst, count, b, step, check, s); \
        else \
            launch_batch_step_t<R, FORMS, RS, HV, false, false, NOISE>(total1, total2, inst, count, b, step, check, s); \
    }
    PHX_BS(true, true)
    PHX_BS(true, false)
    PHX_BS(false, true)
    PHX_BS(false, false)
#undef PHX_BS
    return hipGetLastError();
}

}  // namespace phx
