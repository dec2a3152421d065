// Device code of the streaming whole-step RK4 kernel (one component): all four stages of
// Eqs. rk4_K1-rk4_final in one pass down a band of rows, one wave per strip of columns,
// with no LDS and no barrier.
//
// Lane l of a wave owns W adjacent grid columns (W = 2: complex64 on even widths) from
// column strip*(64 W - 8) - 4 + W l on: the strip's output columns plus a 4-column halo on
// each side, recomputed as in the region kernel; x-neighbours come from DPP wave shifts
// and, with two columns, from the lane's other cell.  The wave walks the rows j = b0-4 ..
// b0+B+3 of its band [b0, b0+B) once; at row j it evaluates
//   stage 1 at row j-1, stage 2 at row j-2, stage 3 at row j-3, stage 4 at row j-4
// (each stage needs its argument at rows r-1..r+1, produced by the stage before it at
// this or an earlier row), and stores the finished row j-4 when it lies in the band.
// (Rows are named for a downward walk; an upward walk mirrors them.)  Odd bands walk
// upwards, so that neighbouring bands reach the 8 rows they both read at the same time
// (the second read is an L2 hit); the stencil is symmetric in y, so the result does not
// depend on the direction.
//
// Per-row inputs (psi, n, P, V) wait in an 8-row ring, loaded 3 rows ahead of their first
// use; the running sums K1 + 2K2 + 2K3 and the stage arguments in rings of 4.  The walk
// runs in chunks of 8 positions, a multiple of every ring length, so every ring slot is a
// fixed register; in the first chunk stage s starts at position 2 s, before which no
// stage needs its rows.  Values that later positions read are pinned where they are formed
// (keep_here).
//
// Where it runs: steps between which something has to happen (noise, the norm of imaginary
// time, small driven grids) and the odd steps of a run; pairs of steps take stream_pair.h.
// On small grids one wave's chain of four stages bounds it (bands of 8 rows, 16 positions:
// 6.5 us per step of the 256^2 trap in imaginary time, 24.6 with bands of 40 rows and a pass
// for the norm), then the VALU issue (imaginary time at 1024^2 24.0 -> 12.9, complex128 27.2
// -> 17.0; drive at 1024^2 26.2 -> 15.9), at 4096^2 HBM (imaginary time 100.7 -> 69; noise,
// drawn in the step, 164 with a pass of its own -> 96 us).
//
// Loads and stores are buffer instructions: the lane's column offset is a constant VGPR
// and the row offset a scalar.  A ghost column (zero x boundary) has an out-of-range offset
// and a ghost row (zero y boundary) reads through an empty descriptor, so both read 0;
// every stage argument is multiplied by 0 in ghost cells and by 1 elsewhere.
#pragma once

#include <type_traits>

#include "philox.h"
#include "stream_wide.h"

namespace phx {

constexpr int step_cols(int w) { return 64 * w - 8; }  // output columns per strip

// Waves per SIMD that the registers allow without scratch memory.
constexpr int step_waves_per_simd(int w, bool f64, bool res, bool drive)
{
    if (w == 1 && !f64) return drive ? 4 : 5;
    return drive || (res && f64) ? 2 : 3;
}

// One band of `B` rows of strip `strip`; `finish(bad, norm)` gets whether a stored value
// is not finite (CHECK; else false without testing: a non-finite value never becomes
// finite again, so testing the last step of a run detects it) and the lane's norm partial.
// IMAG: imaginary time (no reservoir): the derivative is rotated by -i, the input is
// multiplied by `sc`, the scale that restores the previous step's norm, and the norm
// partial is the lane's FP64 sum of |psi_out|^2 over the cells it stores.
// DRIVE: the coherent drive -(i/hbar) E(r) exp(-i omega t_s) joins each stage's
// derivative; E rides in the input ring, the four stage phasors come from a.drive_ph.
// NOISE (W = 2): each stored pair of cells (2p, 2p + 1) first gets its Wiener increment,
// drawn exactly as the separate noise pass draws it (one generator call per pair, the
// reservoir value after the step), so both give the same bits.
template <typename R, int W, bool RES, bool HASV, bool GHOSTS, bool YZERO, bool CHECK, bool IMAG, bool DRIVE, bool NOISE,
          typename F>
__device__ __forceinline__ void stream_band_step(const StepArgs<R>& a, int strip, int band, int B, int dir, R sc,
                                                 uint64_t nstep, F finish)
{
    using C = typename cvec<R>::type;
    static_assert(W == 1 || (W == 2 && sizeof(R) == 4), "two columns per lane: complex64");
    static_assert(!(IMAG && (RES || NOISE || DRIVE)), "imaginary time has no reservoir, noise or drive");
    static_assert(!NOISE || W == 2, "the increments of a cell pair are drawn by one lane");
    constexpr int K = 8;   // rows j - 4 .. j + PF are in flight
    constexpr int PF = 3;  // rows loaded ahead of their first use
    const int lane = threadIdx.x & 63;
    const Coef<R>& c = a.c;
    const int gi = strip * step_cols(W) - 4 + W * lane;  // first column of the lane
    const int ci = wrap_any(gi, a.nx, a.bcx);             // -1: ghost (zero x boundary)
    const bool gcol = GHOSTS && ci < 0;
    const R keep = gcol ? R(0) : R(1);
    const int b0 = band * B;
    const R kdiag = R(2) * (c.ax + c.ay);
    const int rowc = a.nx * (int)sizeof(C), rowr = a.nx * (int)sizeof(R);
    const size_t cells = (size_t)a.nx * a.ny;
    const __amdgpu_buffer_rsrc_t rpi = buffer_of(a.psi_in, cells * sizeof(C));
    const __amdgpu_buffer_rsrc_t rni = buffer_of(a.n_in, RES ? cells * sizeof(R) : 0);
    const __amdgpu_buffer_rsrc_t rP = buffer_of(a.P, RES ? cells * sizeof(R) : 0);
    const __amdgpu_buffer_rsrc_t rV = buffer_of(a.V, HASV ? cells * sizeof(R) : 0);
    const __amdgpu_buffer_rsrc_t rE = buffer_of(a.E, DRIVE ? cells * sizeof(C) : 0);
    const __amdgpu_buffer_rsrc_t rpo = buffer_of(a.psi_out, cells * sizeof(C));
    const __amdgpu_buffer_rsrc_t rno = buffer_of(a.n_out, RES ? cells * sizeof(R) : 0);
    const __amdgpu_buffer_rsrc_t rnull = buffer_of(a.psi_out, 0);  // every access out of range
    const int vc = gcol ? kOutOfRange : (ci < 0 ? 0 : ci) * (int)sizeof(C);
    const int vr = gcol ? kOutOfRange : (ci < 0 ? 0 : ci) * (int)sizeof(R);
    const bool out_col = lane >= 4 / W && lane < 64 - 4 / W && gi < a.nx;
    const int oc = out_col ? gi * (int)sizeof(C) : kOutOfRange;
    const int orr = out_col ? gi * (int)sizeof(R) : kOutOfRange;
    const bool noisy = NOISE && (a.noise_a != R(0) || a.noise_b != R(0));
    double nrm = 0.0;

    // [slot][column of the lane]
    C sp[K][W], sE[K][W], acc[4][W], w[3][4][W];  // w[q]: argument of stage q + 2
    R sn[K][W], sP[K][W], sk[K][W], accn[4][W], wn[3][4][W];
#pragma unroll
    for (int e = 0; e < W; ++e) {
#pragma unroll
        for (int s = 0; s < K; ++s) {
            sp[s][e] = sE[s][e] = czero<C>();
            sn[s][e] = sP[s][e] = R(0);
            sk[s][e] = kdiag;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            acc[s][e] = czero<C>();
            accn[s][e] = R(0);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                w[q][s][e] = czero<C>();
                wn[q][s][e] = R(0);
            }
        }
    }
    C ph[4];
    if constexpr (DRIVE) {
#pragma unroll
        for (int s = 0; s < 4; ++s) ph[s] = a.drive_ph[s];
    }
    // adds -(i/hbar) E ph to (fx, fy)
    auto drive = [&](R& fx, R& fy, const C e, const C p) {
        const R zx = e.x * p.x - e.y * p.y;
        const R zy = e.x * p.y + e.y * p.x;
        fx = fma(c.inv_hbar, zy, fx);
        fy = fma(-c.inv_hbar, zx, fy);
    };

    // The row to fetch advances by one per position: g unwrapped, rw its index under the
    // boundary rule (-1 for a ghost row).  Past the last row of the walk (use == false) rw
    // stays put: the load repeats a row just read and is never used.
    const int npos = B + 8;
    const int start = dir > 0 ? b0 - 4 : b0 + B + 3;
    int g = start;
    int rw = wrap_any(g, a.ny, a.bcy);
    auto load_c = [&](__amdgpu_buffer_rsrc_t r, C (&v)[W], int soff) __attribute__((always_inline)) {
        if constexpr (W == 2) {
            const wf4 x = wload4(r, vc, soff);
            v[0] = C{x.x, x.y};
            v[1] = C{x.z, x.w};
        } else {
            v[0] = buf_load<C>(r, vc, soff);
        }
    };
    auto load_r = [&](__amdgpu_buffer_rsrc_t r, R (&v)[W], int soff) __attribute__((always_inline)) {
        if constexpr (W == 2) {
            const wf2 x = wload2(r, vr, soff);
            v[0] = x.x;
            v[1] = x.y;
        } else {
            v[0] = buf_load<R>(r, vr, soff);
        }
    };
    auto fetch = [&](int s, bool use) __attribute__((always_inline)) {
        const bool grow = YZERO && rw < 0;  // uniform
        const int rr = grow ? 0 : rw;
        load_c(grow ? rnull : rpi, sp[s], rr * rowc);
        if constexpr (DRIVE) load_c(grow ? rnull : rE, sE[s], rr * rowc);
        if (RES) {
            load_r(grow ? rnull : rni, sn[s], rr * rowr);
            load_r(grow ? rnull : rP, sP[s], rr * rowr);
        }
        if (HASV) load_r(grow ? rnull : rV, sk[s], rr * rowr);
        const int gn = g + dir;
        int rn;
        if (YZERO) {
            rn = (gn >= 0 && gn < a.ny) ? gn : -1;
        } else {
            rn = rw + dir;
            rn = rn == a.ny ? 0 : (rn < 0 ? a.ny - 1 : rn);
        }
        g = use ? gn : g;
        rw = use ? rn : rw;
    };
    // the row loaded PF positions ago arrives: scaled (IMAG), V turned into the per-cell
    // constant, and moved out of the register groups that the loads write
    auto arrive = [&](int q) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < W; ++e) {
            if constexpr (IMAG) sp[q][e] = C{sp[q][e].x * sc, sp[q][e].y * sc};
            keep_here(sp[q][e]);
            if constexpr (DRIVE) keep_here(sE[q][e]);
            if (RES) {
                keep_here(sn[q][e]);
                keep_here(sP[q][e]);
            }
            if (HASV) {
                sk[q][e] = fma(c.inv_hbar, sk[q][e], kdiag);
                keep_here(sk[q][e]);
            }
        }
    };
#pragma unroll
    for (int t = 0; t < PF; ++t) fetch(t, true);

    R nf = R(0);  // not 0: a stored value was not finite
    auto positions = [&](auto phase, int base) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(phase)::value;
#pragma unroll
        for (int u = 0; u < K; ++u) {
            const int j = start + dir * (base + u);        // newest row of this position
            fetch(slot<K>(u, -PF), base + u + PF < npos);  // row j + PF
            arrive(slot<K>(u, 0));
#pragma unroll
            for (int s = 1; s <= 4; ++s) {
                if (FIRST && u < 2 * s) continue;
                const int q = slot<K>(u, s), m4 = slot<4>(u, s);  // ring slots of row j - s
                const int r = j - s * dir;
                C cur[W], up[W], dn[W], lr[W];
                R nn[W];
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    cur[e] = s == 1 ? sp[q][e] : w[s - 2][m4][e];
                    up[e] = s == 1 ? sp[slot<K>(u, 2)][e] : w[s - 2][slot<4>(u, s + 1)][e];
                    dn[e] = s == 1 ? sp[slot<K>(u, 0)][e] : w[s - 2][slot<4>(u, s - 1)][e];
                    nn[e] = s == 1 ? sn[q][e] : wn[s - 2][m4][e];
                }
                if constexpr (W == 2) {
                    lr[0] = C{lane_prev(cur[1].x) + cur[1].x, lane_prev(cur[1].y) + cur[1].y};
                    lr[1] = C{cur[0].x + lane_next(cur[0].x), cur[0].y + lane_next(cur[0].y)};
                } else {
                    lr[0] = C{lane_prev(cur[0].x) + lane_next(cur[0].x), lane_prev(cur[0].y) + lane_next(cur[0].y)};
                }
                __builtin_amdgcn_sched_barrier(0);
                const R kk = YZERO ? ((unsigned)r >= (unsigned)a.ny ? R(0) : keep) : keep;
                C y[W];
                R yn[W];
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    R fx, fy, fn;
                    cell_rhs<R, RES, IMAG>(c, cur[e], lr[e].x, lr[e].y, up[e].x + dn[e].x, up[e].y + dn[e].y, nn[e],
                                           sP[q][e], sk[q][e], fx, fy, fn);
                    if constexpr (DRIVE) drive(fx, fy, sE[q][e], ph[s - 1]);
                    C& ac = acc[m4][e];
                    R& an = accn[m4][e];
                    const C p0 = sp[q][e];
                    const R n0 = sn[q][e];
                    if (s < 4) {
                        const R h = s == 3 ? a.dt : a.half_dt;
                        ac = s == 1 ? C{fx, fy} : C{fma(R(2), fx, ac.x), fma(R(2), fy, ac.y)};
                        w[s - 1][m4][e] = C{kk * fma(h, fx, p0.x), kk * fma(h, fy, p0.y)};
                        keep_here(ac);
                        keep_here(w[s - 1][m4][e]);
                        if (RES) {
                            an = s == 1 ? fn : fma(R(2), fn, an);
                            wn[s - 1][m4][e] = kk * fma(h, fn, n0);
                            keep_here(an);
                            keep_here(wn[s - 1][m4][e]);
                        }
                    } else {
                        y[e] = C{fma(a.dt6, ac.x + fx, p0.x), fma(a.dt6, ac.y + fy, p0.y)};
                        if (RES) yn[e] = fma(a.dt6, an + fn, n0);
                    }
                }
                if (s == 4) {
                    // Stores are issued at every position (no branch); a row outside the band
                    // goes to the empty descriptor, whose stores are dropped.
                    const bool st = r >= b0 && r < b0 + B && r < a.ny;  // uniform
                    const int rr = st ? r : 0;
                    if (CHECK) {  // (NOISE: and again where the increment is added; only there: 40 more VGPRs)
                        R t = nf;   // stays 0 while the values are finite
#pragma unroll
                        for (int e = 0; e < W; ++e) {
                            t = fma(y[e].x, R(0), t);
                            t = fma(y[e].y, R(0), t);
                            if (RES) t = fma(yn[e], R(0), t);
                        }
                        nf = st ? t : nf;
                    }
                    if constexpr (NOISE) {
                        if (st && noisy) {
                            const uint32_t pair = (uint32_t)(r * a.nx + gi) >> 1;  // nx and gi even
                            const noise::Philox4 x = noise::philox4x32_10(
                                pair, 0u, (uint32_t)nstep, (uint32_t)(nstep >> 32), a.noise_k0, a.noise_k1);
#pragma unroll
                            for (int e = 0; e < W; ++e)
                                y[e] = noise::add_noise<R, RES>(y[e], RES ? yn[e] : R(0), a.noise_a, a.noise_b,
                                                                x.x[2 * e], x.x[2 * e + 1]);
#pragma unroll
                            for (int e = 0; CHECK && e < W; ++e) nf = fma(y[e].y, R(0), fma(y[e].x, R(0), nf));
                        }
                    }
                    if constexpr (W == 2) {
                        wstore4(wf4{y[0].x, y[0].y, y[1].x, y[1].y}, st ? rpo : rnull, oc, rr * rowc);
                        if (RES) wstore2(wf2{yn[0], yn[1]}, st ? rno : rnull, orr, rr * rowr);
                    } else {
                        buf_store_nt(y[0], st ? rpo : rnull, (int)((unsigned)oc + (unsigned)(rr * rowc)));
                        if (RES) buf_store_nt(yn[0], st ? rno : rnull, (int)((unsigned)orr + (unsigned)(rr * rowr)));
                    }
                    if constexpr (IMAG) {
#pragma unroll
                        for (int e = 0; e < W; ++e)
                            nrm += st && out_col ? (double)y[e].x * y[e].x + (double)y[e].y * y[e].y : 0.0;
                    }
                }
            }
        }
    };
    positions(std::true_type{}, 0);
    for (int base = K; base < npos; base += K) positions(std::false_type{}, base);
    finish(CHECK && out_col && !(nf == R(0)), nrm);
}

}  // namespace phx
