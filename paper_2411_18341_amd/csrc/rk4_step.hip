// Whole-step RK4 kernel: all four stages of Eqs. rk4_K1-rk4_final in one launch.
//
// A workgroup owns a region of 64 columns x H rows of the grid (H = WAVES*ROWS)
// and produces the interior 56 x (H-8) cells: every stage applies the five-point
// stencil once, so after four stages the values are exact up to 4 cells from the
// region edge (the 4-cell halo of the paper's subgrids, Sec. 3.2.4, recomputed
// redundantly instead of exchanged).  The state is read from HBM once (with the
// halo) and written once; the stage arguments, K sums and reservoir values stay in
// registers for the whole step.
//
// Stage s evaluates only the region rows [s, H-s) that the output depends on.
// Lane l of every wave owns region column l; wave w owns rows [w*ROWS, (w+1)*ROWS).
// x-neighbours come from the adjacent lanes by DPP wave shifts, y-neighbours from
// the lane's own registers except at the wave's first and last row, which are
// exchanged through LDS (double-buffered by stage parity: one barrier per stage).
// Region cells outside a zero boundary are ghost cells held at 0 in every stage;
// with a periodic boundary the region wraps.  The output goes to a second state
// buffer (neighbouring regions still read the input's halo).
#include "runtime.h"
#include "step_body.h"

namespace phx {

template <typename R, bool RES, bool HASV, bool GHOSTS, int WAVES, int ROWS>
__global__ __launch_bounds__(WAVES * 64) void rk4_step_kernel(const StepArgs<R> a)
{
    __shared__ typename cvec<R>::type edge[2][WAVES][2][64];
    const bool bad = step_region<R, RES, HASV, GHOSTS, WAVES, ROWS>(a, xcd_tile(blockIdx.x, gridDim.x), edge);
    if (bad) a.flag[0] = 1u;  // benign race: every writer stores 1
}

// GHOSTS: some boundary is zero, so region cells outside the grid must be held at 0
// after every stage; with periodic boundaries in both directions there are none.
template <typename R, bool RES, bool HASV, int WAVES, int ROWS>
static hipError_t launch_step_t(const StepArgs<R>& a, hipStream_t s)
{
    if (a.bcx == PHX_BC_ZERO || a.bcy == PHX_BC_ZERO)
        rk4_step_kernel<R, RES, HASV, true, WAVES, ROWS><<<a.tiles, WAVES * 64, 0, s>>>(a);
    else
        rk4_step_kernel<R, RES, HASV, false, WAVES, ROWS><<<a.tiles, WAVES * 64, 0, s>>>(a);
    return hipGetLastError();
}

// Region shapes (waves per workgroup, rows per wave) instantiated per precision.
// A region of WAVES*ROWS rows yields WAVES*ROWS - 8 output rows; taller regions
// recompute less halo, shorter ones need fewer registers per lane (more waves
// per SIMD).  The first entry is the default; phx_autotune measures them all.
// Shapes {1, B} are the streaming walk with one column per lane and bands of B rows (from 64
// on the height is chosen per grid), {2, B} (and {3, B}, which runs as it) the walk with two columns per lane (complex64,
// even widths), B = 0 choosing the height that fills the device in one wave of workgroups.
static const StepShapeId kFloatShapes[] = {{8, 4}, {16, 4}, {8, 8}, {12, 4}, {12, 6}, {8, 6}, {4, 8}, {16, 6},
                                           {1, 40}, {1, 64}, {1, 88}, {1, 112},
                                           {2, 0}, {2, 40}, {2, 64}, {2, 96}};
static const StepShapeId kDoubleShapes[] = {{8, 4}, {16, 2}, {8, 2}, {12, 4}, {4, 4}, {1, 40}, {1, 64}};

int step_shapes(int precision, const StepShapeId** out)
{
    if (precision == PHX_C64) {
        *out = kFloatShapes;
        return (int)(sizeof(kFloatShapes) / sizeof(kFloatShapes[0]));
    }
    *out = kDoubleShapes;
    return (int)(sizeof(kDoubleShapes) / sizeof(kDoubleShapes[0]));
}

template <typename R, bool RES, bool HASV>
static hipError_t launch_step_shape(const StepShapeId& sh, const StepArgs<R>& a, hipStream_t s)
{
#define PHX_SHAPE(W, K) \
    if (sh.waves == W && sh.rows == K) return launch_step_t<R, RES, HASV, W, K>(a, s)
    if constexpr (sizeof(R) == 4) {
        PHX_SHAPE(8, 4); PHX_SHAPE(16, 4); PHX_SHAPE(8, 8); PHX_SHAPE(12, 4);
        PHX_SHAPE(12, 6); PHX_SHAPE(8, 6); PHX_SHAPE(4, 8); PHX_SHAPE(16, 6);
    } else {
        PHX_SHAPE(8, 4); PHX_SHAPE(16, 2); PHX_SHAPE(8, 2); PHX_SHAPE(12, 4); PHX_SHAPE(4, 4);
    }
#undef PHX_SHAPE
    return hipErrorInvalidValue;
}

bool drive_stream_rows(int rows) { return rows == 40 || rows == 64; }

template <typename R>
hipError_t launch_stream_spinor(bool reservoir, bool has_v, const StepArgs<R>& a, hipStream_t s);

template <typename R>
hipError_t launch_rk4_step(bool reservoir, bool has_v, const StepShapeId& sh, const StepArgs<R>& a,
                           hipStream_t s)
{
    if (a.comps == 2)
        return sh.waves == 1 ? launch_stream_spinor<R>(reservoir, has_v, a, s) : hipErrorInvalidValue;
    if (a.E) return sh.waves == 1 ? launch_step_walk_drive<R>(reservoir, has_v, a, s) : hipErrorInvalidValue;
    if (wide_shape(sh.waves)) {
        if constexpr (sizeof(R) == 4) return launch_step_walk<R, 2>(reservoir, has_v, a, s);
        return hipErrorInvalidValue;
    }
    if (sh.waves == 1) return launch_step_walk<R, 1>(reservoir, has_v, a, s);
    if (reservoir) return has_v ? launch_step_shape<R, true, true>(sh, a, s) : launch_step_shape<R, true, false>(sh, a, s);
    return has_v ? launch_step_shape<R, false, true>(sh, a, s) : launch_step_shape<R, false, false>(sh, a, s);
}

template <typename R>
static hipError_t launch_pair(int columns, bool res, bool hv, const StepArgs<R>& a, hipStream_t s)
{
    if (a.E) return launch_stream_pair_drive<R>(res, hv, a, s);
    if constexpr (sizeof(R) == 4) {
        if (columns == 2) return launch_stream_pair<R, 2>(res, hv, a, s);
    }
    return launch_stream_pair<R, 1>(res, hv, a, s);
}

// Arguments of one whole step (pair > 0: of two) from `src` to `dst` (state buffers) with
// shape sh.
template <typename R>
static StepArgs<R> step_args(const phx_handle* h, const StepShapeId& sh, const void* src, const void* src_n,
                             void* dst, void* dst_n, int parity, int pair = 0)
{
    using C = typename cvec<R>::type;
    const phx_config& c = h->cfg;
    StepArgs<R> a{};
    a.nx = c.nx;
    a.ny = c.ny;
    a.bcx = c.bc_x;
    a.bcy = c.bc_y;
    a.tiles_x = (c.nx + 55) / 56;
    if (pair) {  // two steps per launch, `pair` columns per lane: one wave per band of a strip
        a.tiles_x = pair_strips(c.nx, pair);
        a.band_rows = pair_band_rows(c, pair, h->f.V != nullptr, h->cus);
        a.tiles = a.tiles_x * ((c.ny + a.band_rows - 1) / a.band_rows);
    } else if (c.components == 2) {  // the spinor walk: one wave per band of a strip
        const SpinorPlan p = spinor_plan(c, sh.rows == 64 ? 0 : sh.rows, h->cus);
        a.columns = p.columns;
        a.tiles_x = p.strips;
        a.band_rows = p.band_rows;
        a.tiles = a.tiles_x * ((c.ny + a.band_rows - 1) / a.band_rows);
    } else if (sh.waves <= 3) {  // streaming: one wave per band of a strip
        const StepPlan p = step_plan(c, sh, h->cus);
        a.tiles_x = p.strips;
        a.band_rows = p.band_rows;
        a.tiles = a.tiles_x * ((c.ny + a.band_rows - 1) / a.band_rows);
    } else {
        const int oh = sh.waves * sh.rows - 8;
        a.tiles = a.tiles_x * ((c.ny + oh - 1) / oh);
    }
    a.c = make_coef<R>(c);
    a.half_dt = (R)(0.5 * c.dt);
    a.dt = (R)c.dt;
    a.dt6 = (R)(c.dt / 6.0);
    a.V = (const R*)h->f.V;
    a.P = (const R*)h->f.P;
    a.flag = (unsigned int*)(h->ws + h->L.flag);
    a.psi_in = (const C*)src;
    a.n_in = (const R*)src_n;
    a.psi_out = (C*)dst;
    a.n_out = (R*)dst_n;
    a.comps = c.components;
    if (c.imag_time) {  // buffer b of the partials belongs to state buffer b
        a.imag_slots = (const double*)(h->ws + h->L.imag);
        a.imag_prev = (const double*)(h->ws + h->L.imag_partials) + (parity ? h->L.imag_slots : 0);
        a.imag_partials = (double*)(h->ws + h->L.imag_partials) + (parity ? 0 : h->L.imag_slots);
        a.imag_count = a.tiles <= kImagSelfSum ? a.tiles : 0;
        a.cell_area = c.dx * c.dy;
    }
    if (c.drive) {
        a.E = (const C*)h->f.E;
        a.drive_ph = (const C*)(h->ws + h->L.drive_ph);
    }
    return a;
}

// The noise arguments of a step that draws the increments itself; false if it does not.
template <typename R>
static bool set_noise_args(const phx_config& c, const StepShapeId& sh, const void* step_index, int64_t offset, StepArgs<R>& a)
{
    if (!(c.noise > 0.0) || !noise_in_step(c, sh)) return false;
    a.noise_step = (const uint64_t*)step_index;
    a.noise_offset = offset;
    noise_coefs<R>(c, a.noise_a, a.noise_b, a.noise_k0, a.noise_k1);
    return true;
}

// Trial k of the tuner with shape sh = h->step_shape: one launch and what a step takes beside
// it (the phasors of the drive, the increments of the noise or their pass, the norm of
// imaginary time or its pass).  k = 0 steps the caller's state into the workspace
// copy; later trials alternate between the two workspace copies, so that each one
// reads the state the previous one wrote, as real steps do (a launch that re-read one
// unchanged input would find part of it in the Infinity Cache).  The caller's state
// is never written.  *steps is the number of steps of the trial.
template <typename R>
hipError_t rk4_step_trial(phx_handle* h, const StepShapeId& sh, int k, int* steps)
{
    const phx_config& c = h->cfg;
    const bool res = c.reservoir != 0, hv = h->f.V != nullptr;
    const int pair = pair_columns(c, sh, hv, h->cus);
    *steps = pair ? 2 : 1;
    char* A = h->ws + h->L.alt;
    char* An = res ? h->ws + h->L.alt_n : nullptr;
    char* B = h->ws + h->L.alt2;
    char* Bn = res ? h->ws + h->L.alt2_n : nullptr;
    StepArgs<R> a;
    if (k == 0)
        a = step_args<R>(h, sh, h->f.psi, h->f.n, A, An, 0, pair);
    else if (k & 1)
        a = step_args<R>(h, sh, A, An, B, Bn, 1, pair);
    else
        a = step_args<R>(h, sh, B, Bn, A, An, 0, pair);
    hipError_t e = hipSuccess;
    if (k == 0 && c.imag_time)  // the target, and partials that sum to it for this shape's waves
        e = launch_imag_norm<R>(h, h->f.psi, 0, h->stream);
    if (e == hipSuccess && c.drive) e = launch_drive_phasors<R>(h, 0, *steps, h->stream);
    const bool fused_noise = set_noise_args<R>(c, sh, h->ws + h->L.noise, 0, a);
    if (e == hipSuccess) e = pair ? launch_pair<R>(pair, res, hv, a, h->stream) : launch_rk4_step<R>(res, hv, sh, a, h->stream);
    if (e == hipSuccess && c.imag_time && a.imag_count == 0) e = launch_imag_finish(h, a.imag_partials, a.tiles, h->stream);
    if (e == hipSuccess && c.noise > 0.0 && !fused_noise) e = launch_noise<R>(h, a.psi_out, a.n_out, 0, h->stream);
    return e;
}

template hipError_t rk4_step_trial<float>(phx_handle*, const StepShapeId&, int, int*);
template hipError_t rk4_step_trial<double>(phx_handle*, const StepShapeId&, int, int*);

// Two-step launches among n steps, so that the launches leave the state where n single
// steps would: the n - pairs launches are even in number exactly when n is.
int64_t pair_launches(int64_t n) { return n & 1 ? (n >= 3 ? 2 * ((n + 1) / 4) - 1 : 0) : 2 * (n / 4); }

// Enqueues n whole steps with shape sh on stream s, alternating between the caller's arrays
// (buffer 0) and the workspace copy (buffer 1); h->step_parity is the buffer that
// holds the state before the first of them.  With the two-step form an odd n >= 3 ends
// in the buffer it began in, like an even n.
template <typename R>
phx_status rk4_fused_launches(phx_handle* h, const StepShapeId& sh, int64_t n, hipStream_t s)
{
    const phx_config& c = h->cfg;
    void* S[2] = {h->f.psi, h->ws + h->L.alt};
    void* SN[2] = {h->f.n, c.reservoir ? h->ws + h->L.alt_n : nullptr};
    const bool res = c.reservoir != 0, hv = h->f.V != nullptr;
    const int columns = pair_columns(c, sh, hv, h->cus);
    int64_t pairs = columns ? pair_launches(n) : 0;
    int cur = h->step_parity;
    for (int64_t k = 0, steps = 1; k < n; k += steps) {
        const bool pair = pairs-- > 0;
        steps = pair ? 2 : 1;
        StepArgs<R> a = step_args<R>(h, sh, S[cur], SN[cur], S[cur ^ 1], SN[cur ^ 1], cur, pair ? columns : 0);
        a.check = k + steps == n;  // the wide forms test the last step of the run (values stay non-finite)
        const bool fused_noise = set_noise_args<R>(c, sh, h->ws + h->L.noise, k, a);
        if (c.drive && launch_drive_phasors<R>(h, k, (int)steps, s) != hipSuccess)
            return fail(PHX_EHIP, "drive phasor launch failed");
        hipEvent_t t0 = nullptr;
        hipError_t e = timing_begin(h, &t0);
        if (e == hipSuccess) e = pair ? launch_pair<R>(columns, res, hv, a, s) : launch_rk4_step<R>(res, hv, sh, a, s);
        if (e == hipSuccess) e = timing_end(h, t0, pair ? K_RK4_PAIR : K_RK4_STEP);
        if (e != hipSuccess) return fail(PHX_EHIP, "RK4 step kernel launch: %s", hipGetErrorString(e));
        cur ^= 1;
        if (c.imag_time && a.imag_count == 0) {  // the scale that restores the norm, applied by the next step
            e = timing_begin(h, &t0);
            if (e == hipSuccess) e = launch_imag_finish(h, a.imag_partials, a.tiles, s);
            if (e == hipSuccess) e = timing_end(h, t0, K_IMAG_NORM);
            if (e != hipSuccess) return fail(PHX_EHIP, "imaginary-time norm launch: %s", hipGetErrorString(e));
        }
        if (c.noise > 0.0 && !fused_noise) {
            e = timing_begin(h, &t0);
            if (e == hipSuccess) e = launch_noise<R>(h, S[cur], SN[cur], k, s);
            if (e == hipSuccess) e = timing_end(h, t0, K_NOISE);
            if (e != hipSuccess) return fail(PHX_EHIP, "noise launch: %s", hipGetErrorString(e));
        }
    }
    h->step_parity = cur;
    if (uses_step_index(c) && n > 0 && advance_noise_step(h, n, s) != hipSuccess)
        return fail(PHX_EHIP, "step index advance launch failed");
    return PHX_OK;
}

template phx_status rk4_fused_launches<float>(phx_handle*, const StepShapeId&, int64_t, hipStream_t);
template phx_status rk4_fused_launches<double>(phx_handle*, const StepShapeId&, int64_t, hipStream_t);

// Partials that the waves of the next step sum themselves (0: a pass forms the scale).
int imag_self_sum(const phx_handle* h)
{
    if (!h->cfg.imag_time || h->L.family != PHX_KERNEL_STEP) return 0;
    return h->cfg.precision == PHX_C64 ? step_args<float>(h, h->step_shape, nullptr, nullptr, nullptr, nullptr, 0).imag_count
                                       : step_args<double>(h, h->step_shape, nullptr, nullptr, nullptr, nullptr, 0).imag_count;
}

// n whole steps ending in the caller's arrays.  An odd count first copies the state
// into the workspace and takes one step back (not where two-step launches make the
// number of launches even anyway); the remaining even count alternates (graph replays of
// an even chunk start and end in the caller's arrays).
template <typename R>
phx_status rk4_fused_steps(phx_handle* h, int64_t n)
{
    const phx_config& c = h->cfg;
    const size_t rs = sizeof(R);
    const size_t cells = (size_t)c.nx * c.ny;
    h->step_parity = 0;
    const int G = graph_chunk(c);
    const int64_t direct = h->timing || G == 0 || n < G ? n : n % G;  // steps after the graph replays
    if ((n & 1) && !(pair_columns(c, h->step_shape, h->f.V != nullptr, h->cus) && pair_launches(direct) > 0)) {
        void* alt = h->ws + h->L.alt;
        if (hipMemcpyAsync(alt, h->f.psi, cells * c.components * 2 * rs, hipMemcpyDeviceToDevice, h->stream) !=
                hipSuccess ||
            (c.reservoir && hipMemcpyAsync(h->ws + h->L.alt_n, h->f.n, cells * c.components * rs, hipMemcpyDeviceToDevice,
                                           h->stream) != hipSuccess))
            return fail(PHX_EHIP, "state copy failed");
        h->step_parity = 1;
        phx_status st = rk4_fused_launches<R>(h, n == 1 ? h->lone_shape : h->step_shape, 1, h->stream);
        if (st != PHX_OK) return st;
        --n;
    }
    return rk4_run_graph<R>(h, n);
}

template phx_status rk4_fused_steps<float>(phx_handle*, int64_t);
template phx_status rk4_fused_steps<double>(phx_handle*, int64_t);

}  // namespace phx
