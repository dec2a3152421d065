// One instance of the batched stepper as the kernels see it (the table in the workspace).
#pragma once

#include "phx_kernels.h"

namespace phx {

template <typename R>
struct BatchInst {
    int nx, ny, bcx, bcy;
    int tiles_x, tile0;  // regions across x; first work item of this instance (region form)
    int s_tile0;         // first work item of this instance in the streaming form
    int w_strips;        // wide streaming form (complex64): strips of 120 columns, else 0
    int w_band;          // wide streaming form: rows per band
    int w_tile0;         // first work item of this instance in the wide streaming form
    int p_strips;        // two-step form: strips, rows per band and first work item of this
    int p_band;          // instance in the list of its column count (p_tile0[columns - 1]; in
    int p_tile0[2];      // the other list its range is empty)
    int64_t offset;      // element offset in the packed arrays
    Coef<R> c;
    R half_dt, dt, dt6;
    // Wiener noise: amplitude^2 = noise_a n + noise_b, key, first workgroup of this
    // instance in the noise pass (each instance's cell pairs fill whole workgroups)
    R noise_a, noise_b;
    uint32_t key0, key1;
    int block0;
};

// Two steps per launch over all instances with `columns` columns per lane (batch_pair.h).
template <typename R>
hipError_t launch_batch_pair(int columns, bool res, bool hv, bool ghosts, bool yzero, int total,
                             const BatchInst<R>* inst, int count, const void* pi, const void* ni, void* po, void* no,
                             const void* V, const void* P, unsigned int* flag, bool check, hipStream_t s);
template <typename R, int W>
hipError_t launch_batch_pair_w(bool res, bool hv, bool ghosts, bool yzero, int total, const BatchInst<R>* inst,
                               int count, const void* pi, const void* ni, void* po, void* no, const void* V,
                               const void* P, unsigned int* flag, bool check, hipStream_t s);

}  // namespace phx
