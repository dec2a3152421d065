// Batched whole-step RK4 over many independent one-component instances on grids of
// different sizes, advanced together: the streaming walks, two steps per launch where no
// noise is drawn (batch_pair.h) and one otherwise (batch_walk.h), or one persistent launch
// per step of the region form (a state of 2 GiB, mixed y boundaries).  The region form's
// work list is the concatenation of every instance's regions (56 x (H-8) output cells each,
// H the region height of the step kernel); a workgroup takes items w = blockIdx.x,
// blockIdx.x + gridDim.x, ..., finds the instance by binary search over the instances'
// first item, and runs the same device code as the single-grid whole-step kernel on that
// instance's slice of the packed arrays.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "batch_walk.h"
#include "philox.h"
#include "runtime.h"
#include "step_body.h"
#include "stream_pair.h"

namespace phx {

// Wiener increments of one batched step: one thread per cell pair, each instance's
// pairs in whole workgroups (block_inst maps a workgroup to its instance), the same
// counters and transform as a single-grid handle with the instance's seed.
template <typename R, bool RES>
__global__ __launch_bounds__(256) void batch_noise_kernel(const BatchInst<R>* __restrict__ inst,
                                                          const int* __restrict__ block_inst,
                                                          typename cvec<R>::type* psi, const R* n, uint64_t step)
{
    const BatchInst<R>& I = inst[block_inst[blockIdx.x]];
    if (I.noise_a == (R)0 && I.noise_b == (R)0) return;
    const int64_t p = (int64_t)(blockIdx.x - I.block0) * 256 + threadIdx.x;
    const int64_t q = 2 * p;
    const int64_t cells = (int64_t)I.nx * I.ny;
    if (q >= cells) return;
    const noise::Philox4 x = noise::philox4x32_10((uint32_t)p, 0u, (uint32_t)step, (uint32_t)(step >> 32), I.key0,
                                                  I.key1);
    const int64_t k = I.offset + q;
    noise::noise_pair<R, RES>(psi + k, RES ? n + k : nullptr, q + 1 < cells, (k & 1) == 0, I.noise_a, I.noise_b, x);
}

template <typename R, bool RES, bool HASV, bool GHOSTS, int WAVES, int ROWS>
__global__ __launch_bounds__(WAVES * 64) void batch_step_kernel(
    const BatchInst<R>* __restrict__ inst, int count, int total,
    const typename cvec<R>::type* psi_in, const R* n_in, typename cvec<R>::type* psi_out, R* n_out,
    const R* V, const R* P, unsigned int* flag)
{
    __shared__ typename cvec<R>::type edge[2][WAVES][2][64];
    bool bad = false;
    for (int w = blockIdx.x; w < total; w += gridDim.x) {
        const int t = xcd_tile(w, total);
        int lo = 0, hi = count - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (inst[mid].tile0 <= t) lo = mid; else hi = mid - 1;
        }
        const BatchInst<R>& I = inst[lo];
        StepArgs<R> a;
        a.nx = I.nx;
        a.ny = I.ny;
        a.bcx = I.bcx;
        a.bcy = I.bcy;
        a.tiles_x = I.tiles_x;
        a.tiles = 0;
        a.c = I.c;
        a.half_dt = I.half_dt;
        a.dt = I.dt;
        a.dt6 = I.dt6;
        a.psi_in = psi_in + I.offset;
        a.n_in = RES ? n_in + I.offset : nullptr;
        a.psi_out = psi_out + I.offset;
        a.n_out = RES ? n_out + I.offset : nullptr;
        a.V = HASV ? V + I.offset : nullptr;
        a.P = RES ? P + I.offset : nullptr;
        a.flag = flag;
        bad = step_region<R, RES, HASV, GHOSTS, WAVES, ROWS>(a, t - I.tile0, edge) || bad;
    }
    if (bad) flag[0] = 1u;  // benign race: every writer stores 1
}

// region shape of the batched kernel per precision (8 waves x 4 rows)
constexpr int BW = 8, BR = 4;

// Relative time of a list of `waves` bands that take `positions` each: the issue of the
// busiest SIMD (a single wave reaches 0.82 of the rate), half a wave more for the tail.
static double list_cost(int64_t waves, int positions, int simds)
{
    return positions * (std::max(1.2, (double)waves / simds) + 0.5);
}

constexpr int kFullLists = 6;  // waves per SIMD from which shorter bands cannot help

// Band height of the one-step walk, a multiple of 8 rows evened out over an instance's
// bands; the tallest is the cheapest by list_cost (16 grids of 256^2: bands of 8 rows, 1536
// waves; the step took 31.6 us with bands of 48 and takes 14).  Drawing the increments in
// the step: 128 noisy grids of 256^2, eight steps, 762 us with the separate pass, 562 now.
static int batch_step_band(int ny, int cap)
{
    const int bands = (ny + cap - 1) / cap;
    return ((ny + bands - 1) / bands + 7) / 8 * 8;
}

// Two-step form: columns per lane, strips and band height (up to `cap` rows, evened out
// over the bands where any multiple of 4 will do) of one instance, the column count with the fewer issued
// instructions: strips x bands x positions (B + 16 rows, nine positions' worth of stages left
// out at the start) x instructions per position.
// Tall bands save halo rows, but the last of them end late: up to 56 rows (256 driven grids
// of 128^2 to 1024^2, four steps: 1264 us with bands of up to 44 rows, 1270 with 68, 1304 with 80, 1346
// with 104; 2068 us with one step per launch), fewer where the device would not be full.
// `two`: two columns per lane may be taken (complex64).
static void batch_pair_plan(bool c64, bool two, int nx, int ny, int cap, int* w, int* strips, int* band)
{
    double best = 0.0;
    auto consider = [&](int k, int b) {
        const int n = pair_strips(nx, k);
        const double cost = (double)n * ((ny + b - 1) / b) * (b + 7) * (k == 2 ? 397 : 215);
        if (best == 0.0 || cost < best) {
            best = cost;
            *w = k;
            *strips = n;
            *band = b;
        }
    };
    for (int k = 1; k <= (two && nx % 2 == 0 ? 2 : 1); ++k) {
        const int words = c64 ? k : 2, bands = (ny + cap - 1) / cap;
        if (kPairStep[words] == 4)
            consider(k, pair_band(words, (ny + bands - 1) / bands));
        else
            for (int b = kPairLow[words]; b <= std::max(cap, kPairLow[words]); b += kPairStep[words]) consider(k, b);
    }
}

extern template hipError_t launch_batch_step_forms<float, 1, false>(const BatchForm&, int, int, const BatchInst<float>*, int,
    const BatchState<float>&, uint64_t, bool, hipStream_t);
extern template hipError_t launch_batch_step_forms<double, 1, false>(const BatchForm&, int, int, const BatchInst<double>*, int,
    const BatchState<double>&, uint64_t, bool, hipStream_t);
extern template hipError_t launch_batch_step_forms<float, 3, false>(const BatchForm&, int, int, const BatchInst<float>*, int,
    const BatchState<float>&, uint64_t, bool, hipStream_t);
extern template hipError_t launch_batch_step_forms<float, 3, true>(const BatchForm&, int, int, const BatchInst<float>*, int,
    const BatchState<float>&, uint64_t, bool, hipStream_t);
template hipError_t launch_batch_step_forms<float, 2, false>(const BatchForm&, int, int, const BatchInst<float>*, int,
    const BatchState<float>&, uint64_t, bool, hipStream_t);
template hipError_t launch_batch_step_forms<float, 2, true>(const BatchForm&, int, int, const BatchInst<float>*, int,
    const BatchState<float>&, uint64_t, bool, hipStream_t);

// One launch of a step or a pair of steps over the two lists.
template <typename R>
static hipError_t launch_batch_walk(bool pair, bool noisy, const BatchForm& f, int total1, int total2,
                                    const BatchInst<R>* inst, int count, const BatchState<R>& b, uint64_t step,
                                    bool check, hipStream_t s)
{
    if constexpr (sizeof(R) == 4) {
        if (total2 > 0 && total1 > 0) {
            if (pair) return launch_batch_pair_forms<R, 3>(f, total1, total2, inst, count, b, check, s);
            return noisy ? launch_batch_step_forms<R, 3, true>(f, total1, total2, inst, count, b, step, check, s)
                         : launch_batch_step_forms<R, 3, false>(f, total1, total2, inst, count, b, step, check, s);
        }
        if (total2 > 0) {
            if (pair) return launch_batch_pair_forms<R, 2>(f, 0, total2, inst, count, b, check, s);
            return noisy ? launch_batch_step_forms<R, 2, true>(f, 0, total2, inst, count, b, step, check, s)
                         : launch_batch_step_forms<R, 2, false>(f, 0, total2, inst, count, b, step, check, s);
        }
    }
    if (pair) return launch_batch_pair_forms<R, 1>(f, total1, 0, inst, count, b, check, s);
    return launch_batch_step_forms<R, 1, false>(f, total1, 0, inst, count, b, step, check, s);
}

template <typename R, bool RES, bool HASV, bool GHOSTS>
static hipError_t launch_batch_t(int grid, const BatchInst<R>* inst, int count, int total, const void* pi,
                                 const void* ni, void* po, void* no, const void* V, const void* P,
                                 unsigned int* flag, hipStream_t s)
{
    using C = typename cvec<R>::type;
    batch_step_kernel<R, RES, HASV, GHOSTS, BW, BR><<<grid, BW * 64, 0, s>>>(
        inst, count, total, (const C*)pi, (const R*)ni, (C*)po, (R*)no, (const R*)V, (const R*)P, flag);
    return hipGetLastError();
}

template <typename R>
static hipError_t launch_batch(bool res, bool hv, bool ghosts, int grid, const BatchInst<R>* inst, int count,
                               int total, const void* pi, const void* ni, void* po, void* no, const void* V,
                               const void* P, unsigned int* flag, hipStream_t s)
{
#define PHX_B(RS, HV, G) \
    if (res == RS && hv == HV && ghosts == G) \
        return launch_batch_t<R, RS, HV, G>(grid, inst, count, total, pi, ni, po, no, V, P, flag, s)
    PHX_B(true, false, false); PHX_B(true, true, false); PHX_B(false, false, false); PHX_B(false, true, false);
    PHX_B(true, false, true); PHX_B(true, true, true); PHX_B(false, false, true); PHX_B(false, true, true);
#undef PHX_B
    return hipErrorInvalidValue;
}

struct BatchLayout {
    size_t table, block_inst, alt, alt_n, flag, total;
};

// Workgroups of the noise pass: each instance's cell pairs in whole workgroups of 256.
static int64_t noise_blocks_bound(const phx_batch_desc& d) { return d.total_cells / 512 + d.count + 1; }

static BatchLayout batch_layout(const phx_batch_desc& d)
{
    const size_t rs = d.precision == PHX_C64 ? 4 : 8;
    const size_t inst_bytes = d.precision == PHX_C64 ? sizeof(BatchInst<float>) : sizeof(BatchInst<double>);
    BatchLayout L{};
    size_t off = 0;
    auto take = [&](size_t b) { size_t o = off; off += align_up(b); return o; };
    L.flag = take(256);
    L.table = take((size_t)d.count * inst_bytes);
    L.block_inst = take((size_t)noise_blocks_bound(d) * sizeof(int));
    L.alt = take((size_t)d.total_cells * 2 * rs);
    const bool res = d.params && d.n_params > 0 && d.params[0].reservoir;
    L.alt_n = res ? take((size_t)d.total_cells * rs) : 0;
    L.total = off;
    return L;
}

static phx_status validate_batch(const phx_batch_desc* d)
{
    if (!d) return fail(PHX_EINVAL, "descriptor is NULL");
    if (d->count < 1) return fail(PHX_EINVAL, "count must be >= 1");
    if (d->precision != PHX_C64 && d->precision != PHX_C128) return fail(PHX_EINVAL, "bad precision");
    if (!d->instances || !d->params || d->n_params < 1) return fail(PHX_EINVAL, "instances and params required");
    if (d->check_finite != 0 && d->check_finite != 1) return fail(PHX_EINVAL, "check_finite must be 0 or 1");
    if (d->total_cells < 1 || d->total_cells >= ((int64_t)1 << 40)) return fail(PHX_EINVAL, "bad total_cells");
    if (d->step0 < 0) return fail(PHX_EINVAL, "step0 must be >= 0");
    const int res = d->params[0].reservoir;
    for (int k = 0; k < d->n_params; ++k) {
        phx_config c = d->params[k];
        c.nx = c.ny = 1;
        c.components = 1;
        c.precision = d->precision;
        c.integrator = PHX_RK4;
        c.kernel = PHX_KERNEL_AUTO;
        c.tile_wx = c.tile_rows = 0;
        phx_status s = validate_config(&c);
        if (s != PHX_OK) return s;
        if (c.drive != 0) return fail(PHX_EUNSUPPORTED, "the coherent drive is not implemented for batches");
        if (c.imag_time != 0) return fail(PHX_EUNSUPPORTED, "imaginary time is not implemented for batches");
        if (c.reservoir != res) return fail(PHX_EINVAL, "all params must share the reservoir flag");
    }
    std::vector<std::pair<int64_t, int64_t>> spans;
    spans.reserve(d->count);
    int64_t tiles = 0;
    for (int k = 0; k < d->count; ++k) {
        const phx_instance& I = d->instances[k];
        if (I.nx < 1 || I.ny < 1 || (int64_t)I.nx * I.ny >= ((int64_t)1 << 31))
            return fail(PHX_EINVAL, "instance %d: bad grid %d x %d", k, I.nx, I.ny);
        if (I.param_index < 0 || I.param_index >= d->n_params || I.reserved != 0)
            return fail(PHX_EINVAL, "instance %d: bad param_index or reserved field", k);
        if (I.offset < 0 || I.offset + (int64_t)I.nx * I.ny > d->total_cells)
            return fail(PHX_EINVAL, "instance %d: slice outside the packed arrays", k);
        phx_config c = d->params[I.param_index];
        c.nx = I.nx;
        c.ny = I.ny;
        c.components = 1;
        c.precision = d->precision;
        c.integrator = PHX_RK4;
        c.kernel = PHX_KERNEL_AUTO;
        c.tile_wx = c.tile_rows = 0;
        phx_status s = validate_config(&c);  // stability of dt on this grid
        if (s != PHX_OK) return s;
        spans.push_back({I.offset, I.offset + (int64_t)I.nx * I.ny});
        tiles += (int64_t)((I.nx + 55) / 56) * ((I.ny + BW * BR - 9) / (BW * BR - 8));
    }
    if (tiles >= ((int64_t)1 << 31)) return fail(PHX_EINVAL, "too many work items");
    std::sort(spans.begin(), spans.end());
    for (size_t k = 1; k < spans.size(); ++k)
        if (spans[k].first < spans[k - 1].second) return fail(PHX_EINVAL, "instance slices overlap");
    if (!d->psi || (res && (!d->n || !d->P))) return fail(PHX_EINVAL, "psi (and n, P with the reservoir) required");
    const void* ptrs[] = {d->psi, d->n, d->P, d->V, d->workspace};
    for (const void* p : ptrs)
        if (p && ((uintptr_t)p & 255u)) return fail(PHX_EINVAL, "device pointers must be 256-byte aligned");
    return PHX_OK;
}

// The instance table as the argument of a small launch, which also clears the flag: no copy
// whose source has to outlive the call, so no wait.  Up to kTableLaunches launches; longer
// tables are copied (six launches of 24 or so complex64 instances take what a copy and the
// wait do).  One step of 16 complex128 grids around 128^2: 49.7 us with the copy, 37.2 now; 16
// corrected grids of 256^2 158 -> 137 us per step.
template <typename R>
struct TableChunk {
    static constexpr int N = 3840 / (int)sizeof(BatchInst<R>);
    int first, count;
    BatchInst<R> inst[N];
};
constexpr int kTableLaunches = 6;

template <typename R>
__global__ __launch_bounds__(256) void batch_table_kernel(const TableChunk<R> c, BatchInst<R>* table, unsigned int* flag)
{
    const unsigned int* src = (const unsigned int*)c.inst;
    unsigned int* dst = (unsigned int*)(table + c.first);
    const int words = c.count * (int)(sizeof(BatchInst<R>) / 4);
    for (int k = threadIdx.x; k < words; k += 256) dst[k] = src[k];
    if (c.first == 0 && threadIdx.x < 64) flag[threadIdx.x] = 0u;
}

// Consecutive instances on grids of one size: the band heights are planned once per run (400
// grids of 65^2, one step: 82 us per call with the plan of each, 65 now), and from at most 512
// of many runs (2000 different complex128 grids of 20 to 60 rows, one step: 179 us per call
// with all of them).
struct GridRun {
    int nx, ny, count;
};

template <typename R>
static phx_status batch_run(const phx_batch_desc* d, int64_t n, hipStream_t stream)
{
    const BatchLayout L = batch_layout(*d);
    char* ws = (char*)d->workspace;
    const int res = d->params[0].reservoir;
    std::vector<BatchInst<R>> table(d->count);
    int tile0 = 0;
    std::vector<int> block_inst;
    bool ghosts = false, noisy = false;  // some instance's
    // the streaming forms need every instance's state under 2 GiB (32-bit buffer
    // offsets) and one y boundary rule for all instances
    bool use_stream = true, all_zero_y = true, all_periodic_y = true;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    // tallest bands of the walks: the candidates that give the shortest list; the search ends
    // at once where tall bands already make kFullLists waves per SIMD (45 us of host time for
    // 256 instances), and a walk that the call does not use is not planned
    std::vector<GridRun> runs;
    for (int k = 0; k < d->count; ++k) {
        const phx_instance& I = d->instances[k];
        if (runs.empty() || I.nx != runs.back().nx || I.ny != runs.back().ny)
            runs.push_back(GridRun{I.nx, I.ny, 1});
        else
            ++runs.back().count;
        const phx_config& c = d->params[I.param_index];
        use_stream = use_stream && (double)I.nx * I.ny * 2.0 * sizeof(R) < 2147483648.0 - 256.0;
        all_zero_y = all_zero_y && c.bc_y == PHX_BC_ZERO;
        all_periodic_y = all_periodic_y && c.bc_y == PHX_BC_PERIODIC;
        ghosts = ghosts || c.bc_x == PHX_BC_ZERO || c.bc_y == PHX_BC_ZERO;
        noisy = noisy || c.noise > 0.0;
    }
    use_stream = use_stream && (all_zero_y || all_periodic_y);
    // Pairs of steps where they are built.  Without the reservoir complex128 pairs are still
    // the slower ones on grids whose halos they enlarge too much (64 lanes store 48 columns
    // instead of 56): a position of the pair's walk takes 1.45 times one of the one-step walk,
    // 1.65 times with a potential, so pairs run where their list has so many fewer positions
    // than two of the other (us per step, one / two steps per launch: 2 x 2048^2 48.6 / 45.9,
    // 256 x 200^2 73.6 / 72.3 and with zero boundaries 67.2 / 73.8; with a potential 58.7 /
    // 54.9 and 76.5 / 88.7).
    const bool f64 = sizeof(R) == 8, hasv = d->V != nullptr;
    const bool two = !f64 && batch_pair_built(2, false, res != 0, hasv, ghosts, all_zero_y);
    const bool plan_pairs = use_stream && !noisy && pair_launches(n) > 0 &&
                            batch_pair_built(f64 ? 2 : 1, f64, res != 0, hasv, ghosts, all_zero_y);
    const bool weigh = plan_pairs && f64 && !res;
    const bool plan_steps = !plan_pairs || weigh || 2 * pair_launches(n) < n;
    double s_work = 0.0, p_work = 0.0;  // positions of all items
    const int64_t full = (int64_t)kFullLists * 4 * cus, every = 1 + (int64_t)runs.size() / 256;  // of the runs looked at
    // complex128: 256 noisy grids of 100^2 to 600^2, four steps, 1083 us with bands of up to 64
    // rows, 1045 with 40
    const int s_tallest = f64 ? 40 : 64;
    int s_cap = s_tallest, p_cap = 56;
    double s_best = 0.0, p_best = 0.0;
    for (int cap = s_tallest; plan_steps && cap >= 8; cap -= 8) {
        int64_t waves = 0;
        for (size_t i = 0; i < runs.size(); i += every) {
            const GridRun& g = runs[i];
            const int cols = step_cols(sizeof(R) == 4 && g.nx % 2 == 0 ? 2 : 1), band = batch_step_band(g.ny, cap);
            waves += (int64_t)g.count * ((g.nx + cols - 1) / cols) * ((g.ny + band - 1) / band);
        }
        waves *= every;
        const double cost = list_cost(waves, cap + 4, 4 * cus);
        if (s_best == 0.0 || cost < s_best) {
            s_best = cost;
            s_cap = cap;
        }
        if (waves >= full) break;
    }
    for (int cap = 56; plan_pairs && cap >= 8; cap -= 12) {
        int64_t waves = 0;
        int tallest = 0;
        for (size_t i = 0; i < runs.size(); i += every) {
            const GridRun& g = runs[i];
            int w, strips, band;
            batch_pair_plan(sizeof(R) == 4, two, g.nx, g.ny, cap, &w, &strips, &band);
            waves += (int64_t)g.count * strips * ((g.ny + band - 1) / band);
            tallest = std::max(tallest, band);
        }
        waves *= every;
        const double cost = list_cost(waves, tallest + 7, 4 * cus);
        if (p_best == 0.0 || cost < p_best) {
            p_best = cost;
            p_cap = cap;
        }
        if (waves >= full) break;
    }
    int64_t s_tile0[2] = {0, 0}, p_tile0[2] = {0, 0};  // work items with one and two columns per lane
    int w = 1, p_strips = 1, p_band = 1;
    for (int k = 0; k < d->count; ++k) {
        const phx_instance& I = d->instances[k];
        phx_config c = d->params[I.param_index];
        c.nx = I.nx;
        c.ny = I.ny;
        BatchInst<R>& b = table[k];
        b.nx = I.nx;
        b.ny = I.ny;
        b.bcx = c.bc_x;
        b.bcy = c.bc_y;
        b.tiles_x = (I.nx + 55) / 56;
        b.tile0 = tile0;
        b.offset = I.offset;
        b.c = make_coef<R>(c);
        b.half_dt = (R)(0.5 * c.dt);
        b.dt = (R)c.dt;
        b.dt6 = (R)(c.dt / 6.0);
        tile0 += b.tiles_x * ((I.ny + BW * BR - 9) / (BW * BR - 8));
        // complex64 instances of even width take two columns per lane, the others one
        const int sw = sizeof(R) == 4 && I.nx % 2 == 0 ? 2 : 1;
        b.s_strips = (I.nx + step_cols(sw) - 1) / step_cols(sw);
        b.s_band = batch_step_band(I.ny, s_cap);
        if (plan_pairs && (k == 0 || I.nx != table[k - 1].nx || I.ny != table[k - 1].ny))
            batch_pair_plan(sizeof(R) == 4, two, I.nx, I.ny, p_cap, &w, &p_strips, &p_band);
        b.p_strips = p_strips;
        b.p_band = p_band;
        for (int l = 0; l < 2; ++l) {
            b.s_tile0[l] = (int)std::min<int64_t>(s_tile0[l], INT32_MAX);
            b.p_tile0[l] = (int)std::min<int64_t>(p_tile0[l], INT32_MAX);
        }
        const int64_t s_items = (int64_t)b.s_strips * ((I.ny + b.s_band - 1) / b.s_band);
        const int64_t p_items = (int64_t)b.p_strips * ((I.ny + b.p_band - 1) / b.p_band);
        s_tile0[sw - 1] += s_items;
        p_tile0[w - 1] += p_items;
        s_work += (double)s_items * (b.s_band + 4);
        p_work += (double)p_items * (b.p_band + 7);
        const double scale = c.noise * c.dt / (4.0 * c.dx * c.dy);  // as the single-grid pass forms it
        b.noise_a = (R)(scale * c.R);
        b.noise_b = (R)(scale * c.gamma_c);
        b.key0 = (uint32_t)I.seed;
        b.key1 = (uint32_t)(I.seed >> 32);
    }
    const int total = tile0;
    use_stream = use_stream && s_tile0[0] + s_tile0[1] < INT32_MAX;
    // noise pass over the instances whose step does not draw the increments itself
    for (int k = 0; noisy && k < d->count; ++k) {
        const phx_instance& I = d->instances[k];
        table[k].block0 = (int)block_inst.size();
        if (use_stream && sizeof(R) == 4 && I.nx % 2 == 0) continue;
        const int64_t nb = (((int64_t)I.nx * I.ny + 1) / 2 + 255) / 256;
        block_inst.insert(block_inst.end(), (size_t)nb, k);
    }
    hipError_t e = hipSuccess;
    unsigned int* flag = (unsigned int*)(ws + L.flag);
    constexpr int TN = TableChunk<R>::N;
    // a call that copies and waits for the list of the noise pass anyway copies a longer table
    // too (64 noisy complex128 grids, one step: 156 us with four launches, 145 with the copy)
    const bool by_launch = d->count <= (block_inst.empty() ? kTableLaunches : 1) * TN;
    for (int k = 0; by_launch && k < d->count; k += TN) {
        TableChunk<R> c;
        c.first = k;
        c.count = std::min(TN, d->count - k);
        memcpy(c.inst, table.data() + k, (size_t)c.count * sizeof(BatchInst<R>));
        batch_table_kernel<R><<<1, 256, 0, stream>>>(c, (BatchInst<R>*)(ws + L.table), flag);
        if (e == hipSuccess) e = hipGetLastError();
    }
    if (!by_launch) {
        e = hipMemcpyAsync(ws + L.table, table.data(), table.size() * sizeof(BatchInst<R>), hipMemcpyHostToDevice,
                           stream);
        if (e == hipSuccess) e = hipMemsetAsync(flag, 0, 256, stream);
    }
    if (e == hipSuccess && !block_inst.empty())
        e = hipMemcpyAsync(ws + L.block_inst, block_inst.data(), block_inst.size() * sizeof(int),
                           hipMemcpyHostToDevice, stream);
    // copied host tables go out of scope
    if (e == hipSuccess && (!by_launch || !block_inst.empty())) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return fail(PHX_EHIP, "batch table upload: %s", hipGetErrorString(e));

    // persistent grid of the region form: as many workgroups as fit on the device at once,
    // a multiple of 8 so that every workgroup stays on one XCD's share of the work list
    int grid = 0;
    if (!use_stream) {
        int per_cu = 1;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, batch_step_kernel<R, true, false, false, BW, BR>,
                                                         BW * 64, 0) != hipSuccess || per_cu < 1)
            per_cu = 1;
        grid = std::min(cus * per_cu, (total + 7) / 8 * 8);
        grid = (grid + 7) / 8 * 8;
    }

    const size_t rs = sizeof(R);
    void* S[2] = {d->psi, ws + L.alt};
    void* SN[2] = {d->n, res ? ws + L.alt_n : nullptr};
    int cur = 0;
    // pairs of steps per launch where no increment is drawn in between; then an odd n >= 3
    // ends in the caller's arrays without a copy
    const bool use_pairs = plan_pairs && (!weigh || p_work <= (hasv ? 0.605 : 0.69) * 2.0 * s_work);
    int64_t pairs = use_pairs && use_stream && p_tile0[0] + p_tile0[1] < INT32_MAX ? pair_launches(n) : 0;
    if ((n & 1) && pairs == 0) {
        e = hipMemcpyAsync(S[1], S[0], (size_t)d->total_cells * 2 * rs, hipMemcpyDeviceToDevice, stream);
        if (e == hipSuccess && res)
            e = hipMemcpyAsync(SN[1], SN[0], (size_t)d->total_cells * rs, hipMemcpyDeviceToDevice, stream);
        if (e != hipSuccess) return fail(PHX_EHIP, "batch state copy: %s", hipGetErrorString(e));
        cur = 1;
    }
    const BatchInst<R>* dtab = (const BatchInst<R>*)(ws + L.table);
    for (int64_t k = 0, steps = 1; k < n; k += steps) {
        const bool pair = pairs-- > 0;
        steps = pair ? 2 : 1;
        const bool check = k + steps == n;
        if (use_stream) {
            using C = typename cvec<R>::type;
            const BatchForm form{res != 0, d->V != nullptr, ghosts, all_zero_y};
            const BatchState<R> b{(const C*)S[cur], (const R*)SN[cur], (C*)S[cur ^ 1], (R*)SN[cur ^ 1],
                                  (const R*)d->V, (const R*)d->P, flag};
            e = launch_batch_walk<R>(pair, noisy, form, (int)(pair ? p_tile0[0] : s_tile0[0]),
                                     (int)(pair ? p_tile0[1] : s_tile0[1]), dtab, d->count, b, (uint64_t)(d->step0 + k),
                                     check, stream);
        } else
            e = launch_batch<R>(res != 0, d->V != nullptr, ghosts, grid, dtab, d->count, total, S[cur], SN[cur],
                                S[cur ^ 1], SN[cur ^ 1], d->V, d->P, flag, stream);
        if (e != hipSuccess) return fail(PHX_EHIP, "batch step launch: %s", hipGetErrorString(e));
        cur ^= 1;
        if (!block_inst.empty()) {
            using C = typename cvec<R>::type;
            const unsigned blocks = (unsigned)block_inst.size();
            const int* bi = (const int*)(ws + L.block_inst);
            const uint64_t step = (uint64_t)(d->step0 + k);
            if (res)
                batch_noise_kernel<R, true><<<blocks, 256, 0, stream>>>(dtab, bi, (C*)S[cur], (const R*)SN[cur],
                                                                        step);
            else
                batch_noise_kernel<R, false><<<blocks, 256, 0, stream>>>(dtab, bi, (C*)S[cur], nullptr, step);
            e = hipGetLastError();
            if (e != hipSuccess) return fail(PHX_EHIP, "batch noise launch: %s", hipGetErrorString(e));
        }
    }
    if (d->check_finite) {
        unsigned int v = 0;
        e = hipMemcpyAsync(&v, flag, sizeof(v), hipMemcpyDeviceToHost, stream);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
        if (e != hipSuccess) return fail(PHX_EHIP, "batch flag read: %s", hipGetErrorString(e));
        if (v) return fail(PHX_ENONFINITE, "a non-finite value appeared in the batch");
    }
    return PHX_OK;
}

}  // namespace phx

using namespace phx;

phx_status phx_batch_workspace_bytes(const phx_batch_desc* desc, size_t* out)
{
    clear_error();
    if (!out) return fail(PHX_EINVAL, "out is NULL");
    phx_status s = validate_batch(desc);
    if (s != PHX_OK) return s;
    *out = batch_layout(*desc).total;
    return PHX_OK;
}

phx_status phx_batch_step(const phx_batch_desc* desc, int64_t n_steps, void* hip_stream)
{
    clear_error();
    phx_status s = validate_batch(desc);
    if (s != PHX_OK) return s;
    if (n_steps < 0) return fail(PHX_EINVAL, "n_steps must be >= 0");
    const BatchLayout L = batch_layout(*desc);
    if (!desc->workspace || desc->workspace_bytes < L.total)
        return fail(PHX_EWORKSPACE, "workspace of %zu bytes needed", L.total);
    if (n_steps == 0) return PHX_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    return desc->precision == PHX_C64 ? batch_run<float>(desc, n_steps, st) : batch_run<double>(desc, n_steps, st);
}
