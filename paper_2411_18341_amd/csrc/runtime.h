// Host-side internals of libphx shared by the runtime translation units: error
// reporting, workspace layout, tile plans, coefficient formation and the handle.
#pragma once

#include <stddef.h>

#include <vector>

#include "phx_kernels.h"

namespace phx {

// Region shape of the whole-step RK4 kernel: waves per workgroup, rows per wave.
struct StepShapeId {
    int waves, rows;
};
inline bool operator==(const StepShapeId& a, const StepShapeId& b) { return a.waves == b.waves && a.rows == b.rows; }
inline bool operator!=(const StepShapeId& a, const StepShapeId& b) { return !(a == b); }

struct TilePlan {
    TileShape ts;
    int tiles_x;
    int tiles;
};

// Byte offsets of the workspace regions of one handle (all 256-byte aligned).
struct Layout {
    size_t flag;        // non-finite flag word(s)
    size_t obs;         // OBS_SLOTS doubles: reduced observables
    size_t partials;    // obs_blocks * OBS_SLOTS doubles
    size_t y[2], yn[2]; // RK4 stage arguments (ping-pong)
    size_t acc, accn;   // RK4 running sum K1 + 2 K2 + 2 K3
    size_t k[7];        // Dormand-Prince stage derivatives
    size_t ys;          // Dormand-Prince stage argument
    size_t alt;         // second state buffer for psi (whole-step RK4, Dormand-Prince)
    size_t alt_n;       // second state buffer for n (whole-step RK4)
    size_t alt2, alt2_n;  // third state buffer (whole-step RK4: the tuner's trial launches)
    size_t noise;       // uint64 index of the next step, read by the noise and the drive
                        // (allocated when either is on)
    size_t drive_ph;    // RK4 with drive: the stage phasors of one launch (up to two steps)
    size_t imag;        // imaginary time: [0] target norm of the call, [1] restoring scale
    size_t imag_partials;  // imaginary time: two arrays of imag_slots norm partials
    size_t imag_slots;
    int family;         // PHX_KERNEL_STAGE or PHX_KERNEL_STEP for RK4
    size_t err;         // Dormand-Prince error partials
    int obs_blocks;
    int err_blocks;
    TilePlan tiles;
    size_t total;
};

phx_status fail(phx_status s, const char* fmt, ...);
void clear_error();
const char* last_error();
size_t align_up(size_t x);
phx_status validate_config(const phx_config* c);
Layout make_layout(const phx_config& c);
TilePlan plan_tiles(int nx, int ny, int wx, int rows);
bool valid_step_shape(int precision, int waves, int rows);
template <typename R> Coef<R> make_coef(const phx_config& c);

}  // namespace phx

struct phx_handle {
    phx_config cfg;
    phx_fields f;
    hipStream_t stream;
    phx::Layout L;
    char* ws;
    phx_info info;
    double* host;           // pinned: [0, OBS_SLOTS) observables, [OBS_SLOTS] flag word,
                            // [OBS_SLOTS + 1] error norm
    hipEvent_t flag_ready;  // recorded after the flag read-back of the last phx_step
    bool flag_pending;
    // Dormand-Prince: where the current state lives (the caller's psi or the
    // workspace copy) and whether K1 = f(state) is valid in k[fsal].
    void* cur;
    void* other;
    void* cur_n;
    void* other_n;
    phx::StepShapeId step_shape;  // whole-step RK4 shape in use
    phx::StepShapeId lone_shape;  // the shape for a call of one step
    int cus;                      // compute units of the handle's device
    phx::TilePlan stage_tiles;    // stage-fused RK4 tile plan in use
    int step_parity;              // whole-step family: buffer holding the state (0 = caller's)
    // coherent drive: time and step index of the last phx_create / phx_set_info
    double drive_t0;
    int64_t drive_k0;
    int fsal;               // index of the buffer that holds K1 of the current state
    bool k1_valid;
    // attempt log of the caller (phx_log_attempts): (dt, err, accepted) per attempt
    double* att_log;
    int64_t att_cap;
    int64_t* att_count;
    // hipGraph of graph_steps RK4 steps, captured on cap_stream, replayed on stream
    hipStream_t cap_stream;
    hipGraphExec_t graph;
    bool graph_dirty;
    // kernel timing (phx_set_timing / phx_kernel_times)
    struct TimedLaunch {
        hipEvent_t start, stop;
        int kind;
    };
    bool timing;
    std::vector<hipEvent_t> free_events;
    std::vector<TimedLaunch> pending;
    double kind_ms[PHX_MAX_KERNEL_KINDS];
    int64_t kind_launches[PHX_MAX_KERNEL_KINDS];
};

namespace phx {
// Kernel kinds for phx_kernel_times; names in kernel_kind_name().
enum KernelKind {
    K_RK4_S1 = 0, K_RK4_S2, K_RK4_S3, K_RK4_S4, K_OBS, K_DP_S1, K_DP_S2, K_DP_S3, K_DP_S4,
    K_DP_S5, K_DP_S6, K_DP_S7, K_DP_ERR, K_BATCH, K_RK4_STEP, K_NOISE, K_IMAG_NORM, K_IMAG_SCALE, K_RK4_PAIR, K_KINDS_
};
const char* kernel_kind_name(int k);
// Timing brackets around one launch (no-ops unless timing is on).
hipError_t timing_begin(phx_handle* h, hipEvent_t* start);
hipError_t timing_end(phx_handle* h, hipEvent_t start, int kind);
const void* state_psi(const phx_handle* h);
// Observables: kernel arguments from a configuration, its tile plan and the fields
// (drive phase at time t), and phx_obs from the reduced slots.
template <typename R>
ObsArgs<R> obs_args(const phx_config& c, const TilePlan& tiles, const void* psi, const void* n, const void* V,
                    const void* P, const void* E, double t, double* partials, double* out);
void obs_from_slots(const phx_config& c, const double* q, phx_obs* out);
const void* state_n(const phx_handle* h);
phx_status create_rk45(phx_handle* h);
// Whole-attempt Dormand-Prince walk (dp_walk.h).
template <typename R> struct DpWalkArgs;
template <typename R, int COMPS> hipError_t launch_dp_walk(bool res, const DpWalkArgs<R>& a, hipStream_t s);
template <typename R> phx_status rk4_fused_steps(phx_handle* h, int64_t n);
template <typename R> phx_status rk4_fused_launches(phx_handle* h, const StepShapeId& sh, int64_t n, hipStream_t s);
template <typename R> phx_status rk4_stage_launches(phx_handle* h, int64_t n, hipStream_t s);
int graph_chunk(const phx_config& c);
template <typename R> phx_status rk4_run_graph(phx_handle* h, int64_t n);
template <typename R> hipError_t rk4_step_trial(phx_handle* h, const StepShapeId& sh, int k, int* steps);
template <typename R> hipError_t rk4_stage_trial(phx_handle* h, const TileShape& ts);
int step_shapes(int precision, const StepShapeId** out);
bool step_shape_fits(const phx_config& c, int waves);
// A whole-step shape this configuration can run (size limit of the streaming form;
// imaginary time, the drive and the spinor only on streaming shapes, the drive and
// the spinor on bands of 40 and 64 rows).
bool step_shape_allowed(const phx_config& c, const StepShapeId& sh);
bool drive_stream_rows(int rows);
// Streaming forms (stream_step.h): shapes {1, B} with one column per lane, {2, B} and {3, B}
// with two; strips and band height for this grid on a device with `cus` compute units.
template <typename R> struct StepArgs;
bool wide_shape(int waves);
struct StepPlan {
    int strips, band_rows;
};
StepPlan step_plan(const phx_config& c, const StepShapeId& sh, int cus);
template <typename R, int W>
hipError_t launch_step_walk(bool reservoir, bool has_v, const StepArgs<R>& a, hipStream_t s);
template <typename R>
hipError_t launch_step_walk_drive(bool reservoir, bool has_v, const StepArgs<R>& a, hipStream_t s);

// Band height of a walk that is bound by its VALU issue: of the heights with which every
// wave (one per band of a strip) is resident at once, the one whose busiest SIMD ends first.
// A wave walks rows + halo positions, `skipped` of them without work; heights are
// lo + k step.  One and two waves on a SIMD issue at the shares `one` and `two` of its rate,
// measured on the two-step walk: one wave 0.82 (63.6 us per step at 4096^2 with bands of 152
// rows, against 59.4 with two waves and bands of 80), two 0.97.
struct BandFill {
    int rows;
    double cost;  // positions times waves on the busiest SIMD, over the issue rate
};
inline BandFill band_fill(int strips, int ny, int halo, int skipped, int lo, int step, int cus, int waves_per_simd,
                          double one = 0.82, double two = 0.97)
{
    const int simds = 4 * (cus > 0 ? cus : 256);
    BandFill best{0, 0.0};
    for (int n = 1; n <= waves_per_simd; ++n) {
        const int bands = simds * n / strips;
        if (bands < 1 && n < waves_per_simd) continue;
        const int need = bands < 1 ? ny : (ny + bands - 1) / bands;
        const int rows = need <= lo ? lo : lo + (need - lo + step - 1) / step * step;
        const int64_t waves = (int64_t)strips * ((ny + rows - 1) / rows);
        const int busy = (int)((waves + simds - 1) / simds);
        const double rate = busy == 1 ? one : (busy == 2 ? two : 1.0);
        const double cost = busy * (double)(rows + halo - skipped) / rate;
        if (best.rows == 0 || cost < best.cost) best = BandFill{rows, cost};
    }
    return best;
}
// Two steps per launch of the streaming forms (stream_pair.h): the columns per lane with
// which shape sh runs this way for this configuration (0: it takes single steps), the
// strips and the band height.
int pair_columns(const phx_config& c, const StepShapeId& sh, bool has_v, int cus);
StepShapeId default_step_shape(const phx_config& c);
StepShapeId default_lone_shape(const phx_config& c);
int pair_strips(int nx, int w);
// With the reservoir, a potential and a zero boundary, pairs of two complex64 columns or one
// complex128 column per lane (words = 2) run one wave per SIMD and are slower than single
// steps at every size: us per step, one / two steps per launch, complex64 10.7 / 15.2 at
// 1024^2, 55 / 62 at 3000^2, 105 / 108 at 4096^2; complex128 16.4 / 21.4, 118 / 115 and
// 211 / 226.  Pairs with one complex64 column per lane (words = 1) take 11.9, 55 and 86.
constexpr bool pair_pays(int words, bool res, bool has_v, bool ghosts)
{
    return words == 1 || !(res && has_v && ghosts);
}
int64_t pair_launches(int64_t n);  // two-step launches among n steps
// Columns per lane, strips and band height of the spinor walk (stream_spinor.h).
struct SpinorPlan {
    int columns, strips, band_rows;
};
SpinorPlan spinor_plan(const phx_config& c, int rows, int cus);
int pair_band_rows(const phx_config& c, int w, bool has_v, int cus);
template <typename R, int W>
hipError_t launch_stream_pair(bool reservoir, bool has_v, const StepArgs<R>& a, hipStream_t s);
template <typename R>
hipError_t launch_stream_pair_drive(bool reservoir, bool has_v, const StepArgs<R>& a, hipStream_t s);
int rk4_family(const phx_config& c);
phx_status step_rk45(phx_handle* h, int64_t n, phx_info* out);
phx_status set_info_rk45(phx_handle* h, const phx_info* in);
// Wiener increment of one step on (psi, n) with step index base + offset; the base
// is advanced after each run of steps and set at creation and by phx_set_info.
template <typename R> hipError_t launch_noise(const phx_handle* h, void* psi, const void* n, int64_t offset,
                                              hipStream_t s);
hipError_t advance_noise_step(const phx_handle* h, int64_t by, hipStream_t s);
// The increment's variance a n + b (a = nu R dt / (4 dV), b = nu gamma_c dt / (4 dV),
// formed in double) and the generator key (the seed's two words).
template <typename R>
inline void noise_coefs(const phx_config& c, R& a, R& b, uint32_t& k0, uint32_t& k1)
{
    const double scale = c.noise * c.dt / (4.0 * c.dx * c.dy);
    a = (R)(scale * c.R);
    b = (R)(scale * c.gamma_c);
    k0 = (uint32_t)c.seed;
    k1 = (uint32_t)(c.seed >> 32);
}
// The two-column step adds the increment itself before its final store (one
// component, complex64, even widths); elsewhere a separate pass follows the step.
bool noise_in_step(const phx_config& c, const StepShapeId& sh);
hipError_t set_noise_step(const phx_handle* h, int64_t value, hipStream_t s);
// Drive phasors exp(-i omega t_s) of the four RK4 stage times of the `steps` (1 or 2) steps
// from index base + offset on, written to the workspace (one thread; graph-replay safe).
template <typename R> hipError_t launch_drive_phasors(const phx_handle* h, int64_t offset, int steps, hipStream_t s);
bool uses_step_index(const phx_config& c);
// Imaginary time: deterministic total norm of psi into the target (mode 0) or the
// restoring scale (mode 1), and the pointwise scale pass.
int imag_norm_blocks(int64_t M);
template <typename R> hipError_t launch_imag_norm(const phx_handle* h, const void* psi, int mode, hipStream_t s);
template <typename R> hipError_t launch_imag_scale(const phx_handle* h, void* psi, hipStream_t s);
// Imaginary time, streaming forms: the restoring scale from `count` per-wave partials.  Up to
// kImagSelfSum partials are summed by every wave of the next step itself, a few loads per
// lane instead of a launch (256^2, 160 waves: 6.5 us per step; the launch alone took 4.5; 1024^2, about
// 2400 waves: 13.7 summed by the waves, 12.3 with the launch).
constexpr int kImagSelfSum = 512;
int imag_self_sum(const phx_handle* h);
hipError_t launch_imag_finish(const phx_handle* h, const double* partials, int count, hipStream_t s);
}  // namespace phx
