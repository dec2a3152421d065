// One instance of the batched stepper as the kernels see it (the table in the workspace).
#pragma once

#include "phx_kernels.h"
#include "runtime.h"

namespace phx {

template <typename R>
struct BatchInst {
    int nx, ny, bcx, bcy;
    int tiles_x, tile0;  // regions across x; first work item of this instance (region form)
    int s_strips;        // one-step walk: strips, rows per band and first work item of this
    int s_band;          // instance in the list of its column count (s_tile0[columns - 1]; in
    int s_tile0[2];      // the other list its range is empty)
    int p_strips;        // the same of the two-step walk
    int p_band;
    int p_tile0[2];
    int64_t offset;      // element offset in the packed arrays
    Coef<R> c;
    R half_dt, dt, dt6;
    // Wiener noise: amplitude^2 = noise_a n + noise_b, key, first workgroup of this
    // instance in the noise pass (each instance's cell pairs fill whole workgroups)
    R noise_a, noise_b;
    uint32_t key0, key1;
    int block0;
};

// The packed arrays of one launch, and the terms that all instances share.
template <typename R>
struct BatchState {
    const typename cvec<R>::type* psi_in;
    const R* n_in;
    typename cvec<R>::type* psi_out;
    R* n_out;
    const R *V, *P;
    unsigned int* flag;
};
struct BatchForm {
    bool res, hasv, ghosts, yzero;  // yzero: every instance has a zero y boundary, else none
};

// Variants whose pairs of steps are built (and run, see batch_run); words as in pair_pays.
// In complex128 a potential leaves registers for one wave per SIMD with the reservoir or a
// zero y boundary, and the pairs are slower than single steps: us per step, one / two steps
// per launch, 256 grids of 200^2: with the reservoir 138 / 179, zero boundaries 126 / 199,
// without the reservoir and zero in y 73 / 99.
constexpr bool batch_pair_built(int words, bool f64, bool res, bool hasv, bool ghosts, bool yzero)
{
    return f64 ? !(hasv && (res || yzero)) : pair_pays(words, res, hasv, ghosts);
}

// One step (batch_walk.h) or two (batch_pair.h) over all instances in one launch: total1
// items with one column per lane, total2 with two.  FORMS: 1, 2, or 3 where both occur.
template <typename R, int FORMS, bool NOISE>
hipError_t launch_batch_step_forms(const BatchForm& f, int total1, int total2, const BatchInst<R>* inst, int count,
                                   const BatchState<R>& b, uint64_t step, bool check, hipStream_t s);
template <typename R, int FORMS>
hipError_t launch_batch_pair_forms(const BatchForm& f, int total1, int total2, const BatchInst<R>* inst, int count,
                                   const BatchState<R>& b, bool check, hipStream_t s);

}  // namespace phx
