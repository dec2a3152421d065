// Device code of the two-step streaming RK4 kernel (one component): two whole steps of
// Eqs. rk4_K1-rk4_final in one pass over the state.
//
// The band walk of stream_step.h (W = 2 grid columns per lane: complex64 on even widths;
// W = 1: complex128, odd widths, the drive) with eight stages in the pipeline instead of
// four: at row j the stages of the first step run at rows j - 1 ..
// j - 4 and finish row j - 4 of the state in between, which stays in registers; the
// stages of the second step run at rows j - 5 .. j - 8 on it, and row j - 8 is stored.
// The state thus moves through HBM once for two steps.  The halo doubles: 8 columns on
// each side (112 output columns per strip of 128, 48 of 64) and B + 16 rows for B output rows.
// The arithmetic per cell and its order are those of the other whole-step forms, so the
// results agree bit for bit with two single steps.
//
// Stage k = 1..8 of the pipeline starts at position 2 k: no stage after it needs its
// earlier rows.  The first twelve positions are a copy of the loop body with the stages
// left out that have not started.  The walk runs in whole chunks (an exit inside a
// chunk costs 30 to 70 registers) except with one complex64 column, which leaves registers
// for it: that walk ends at a multiple of four positions, inside a chunk by ending the
// program there (a branch to a common end would make every ring slot live to it).
//
// Bound by the VALU issue: 24.8 instructions per cell and stage, and with the halo (128 x
// (B + 10) cells evaluated for 112 x B stored) all SIMDs issue back to back: 118.8 us per
// launch, 59.4 us per step, at 4096^2 driven (B 80, 1924 waves, 2 per SIMD); the one-step
// wide form takes 92.8 us per step, bound by HBM (28 bytes per point and step).  One
// wave per SIMD with bands of 152 rows takes 63.6 us, ragged fillings 66 to 95 us.  One
// complex64 column: with heights of any multiple of 4 rows 9.0 us per step at 1024^2, 13.7 at
// 1536^2 and 20.9 at 2047^2; in whole chunks 11.9, 16.2 and 22.7.
#pragma once

#include <type_traits>

#include "stream_wide.h"

namespace phx {

// Waves per SIMD that the registers allow without scratch memory; words = 32-bit words of
// the lane's real values per row (2: two complex64 columns or one complex128 column).
constexpr int pair_waves_per_simd(int words, bool res, bool hasv, bool ghosts, bool drive)
{
    if (drive) return words == 1 ? 2 : 1;
    if (words == 1) return res && hasv ? 3 : 4;
    return res ? (hasv ? 1 : 2) : (hasv || ghosts ? 2 : 3);
}

constexpr int kPairHalo = 8;
constexpr int pair_cols(int w) { return 64 * w - 2 * kPairHalo; }  // output columns per strip
// Band heights whose positions the walk does not idle through, low + k step by `words` (as
// above), and the smallest of at least `rows`.
constexpr int kPairLow[3] = {0, 8, 20}, kPairStep[3] = {0, 4, 12};
constexpr int pair_band(int words, int rows)
{
    const int lo = kPairLow[words], step = kPairStep[words];
    return rows <= lo ? lo : lo + (rows - lo + step - 1) / step * step;
}

// One band of `B` rows of strip `strip`; `finish(bad)` gets whether a stored value is not
// finite (CHECK; else false without testing).  DRIVE: the coherent drive joins each stage's
// derivative; a.drive_ph holds the eight phasors of the two steps.
template <typename R, int W, bool RES, bool HASV, bool GHOSTS, bool YZERO, bool CHECK, bool DRIVE, typename F>
__device__ __forceinline__ void stream_band_pair(const StepArgs<R>& a, int strip, int band, int B, int dir, F finish)
{
    using C = typename cvec<R>::type;
    static_assert(W == 1 || (W == 2 && sizeof(R) == 4), "two columns per lane: complex64");
    constexpr int K = 12;  // rows j - 8 .. j + PF of the inputs are in flight
    constexpr int PF = RES && HASV ? 2 : 3;  // rows loaded ahead of their first use
    const int lane = threadIdx.x & 63;
    const Coef<R>& c = a.c;
    const int gi = strip * pair_cols(W) - kPairHalo + W * lane;  // first column of the lane
    const int ci = wrap_any(gi, a.nx, a.bcx);                     // -1: ghost (zero x boundary)
    const bool gcol = GHOSTS && ci < 0;
    R keep = gcol ? R(0) : R(1);
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
    const bool out_col = lane >= kPairHalo / W && lane < 64 - kPairHalo / W && gi < a.nx;
    const int oc = out_col ? gi * (int)sizeof(C) : kOutOfRange;
    const int orr = out_col ? gi * (int)sizeof(R) : kOutOfRange;

    // [step][slot][cell of the lane]; step 0 reads the input, step 1 the state in between
    C sp[2][K][W], acc[2][4][W], w[2][3][3][W];  // w[.][q]: argument of stage q + 2
    R sn[2][K][W], accn[2][4][W], wn[2][3][3][W];
    R sP[K][W], sk[K][W];
    C sE[K][W];
#pragma unroll
    for (int e = 0; e < W; ++e) {
#pragma unroll
        for (int s = 0; s < K; ++s) {
            sP[s][e] = R(0);
            sE[s][e] = czero<C>();
            sk[s][e] = kdiag;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int s = 0; s < K; ++s) {
                sp[h][s][e] = czero<C>();
                sn[h][s][e] = R(0);
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                acc[h][s][e] = czero<C>();
                accn[h][s][e] = R(0);
            }
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int s = 0; s < 3; ++s) {
                    w[h][q][s][e] = czero<C>();
                    wn[h][q][s][e] = R(0);
                }
        }
    }

    C ph[8];
    if constexpr (DRIVE) {
#pragma unroll
        for (int s = 0; s < 8; ++s) ph[s] = a.drive_ph[s];
    }

    const int npos = B + 2 * kPairHalo;
    const int start = dir > 0 ? b0 - kPairHalo : b0 + B - 1 + kPairHalo;
    int g = start;
    int rw = wrap_any(g, a.ny, a.bcy);
    auto fetch = [&](int s, bool use) __attribute__((always_inline)) {
        const bool grow = YZERO && rw < 0;  // uniform: a ghost row reads 0 through the empty descriptor
        const int rr = grow ? 0 : rw;
        auto load_complex = [&](__amdgpu_buffer_rsrc_t r, C (&v)[W]) __attribute__((always_inline)) {
            if constexpr (W == 2) {
                const wf4 x = wload4(r, vc, rr * rowc);
                v[0] = C{x.x, x.y};
                v[1] = C{x.z, x.w};
            } else {
                v[0] = buf_load<C>(r, vc, rr * rowc);
            }
        };
        load_complex(grow ? rnull : rpi, sp[0][s]);
        if constexpr (DRIVE) load_complex(grow ? rnull : rE, sE[s]);
        auto load_real = [&](__amdgpu_buffer_rsrc_t r, R (&v)[W]) __attribute__((always_inline)) {
            if constexpr (W == 2) {
                const wf2 x = wload2(r, vr, rr * rowr);
                v[0] = x.x;
                v[1] = x.y;
            } else {
                v[0] = buf_load<R>(r, vr, rr * rowr);
            }
        };
        if (RES) {
            load_real(grow ? rnull : rni, sn[0][s]);
            load_real(grow ? rnull : rP, sP[s]);
        }
        if (HASV) {
            R v[W];
            load_real(grow ? rnull : rV, v);
#pragma unroll
            for (int e = 0; e < W; ++e) sk[s][e] = fma(c.inv_hbar, v[e], kdiag);
        }
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
#pragma unroll
    for (int t = 0; t < PF; ++t) fetch(t, true);

    R nf = R(0);
    auto positions = [&](auto phase, int base) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(phase)::value;
#pragma unroll
        for (int u = 0; u < K; ++u) {
            const int j = start + dir * (base + u);        // newest row of this position
            fetch(slot<K>(u, -PF), base + u + PF < npos);  // row j + PF
            if constexpr (DRIVE && sizeof(R) == 8 && RES && GHOSTS) {
                park(keep);
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    park(ph[s].x);
                    park(ph[s].y);
                }
            }
            // Row j arrives: its values leave the four- and two-register groups that the
            // loads write (kept there for their whole life they fragment the register file).
#pragma unroll
            for (int e = 0; e < W; ++e) {
                const int q = slot<K>(u, 0);
                keep_here(sp[0][q][e]);
                if (RES) {
                    keep_here(sn[0][q][e]);
                    keep_here(sP[q][e]);
                }
                if (HASV) keep_here(sk[q][e]);
                if constexpr (DRIVE) keep_here(sE[q][e]);
            }
#pragma unroll
            for (int k = 1; k <= 8; ++k) {
                if (FIRST && u < 2 * k) continue;
                const int h = (k - 1) / 4, s = (k - 1) % 4 + 1;  // step and its stage
                const int q = slot<K>(u, k);                     // ring slot of row j - k
                const int m = slot<3>(u, k), a4 = slot<4>(u, k);
                const int r = j - k * dir;
                // argument rows: the state itself in stage 1, else the stage argument
                C cur[W], up[W], dn[W], lr[W];
                R nn[W];
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    if (s == 1) {
                        cur[e] = sp[h][q][e];
                        up[e] = sp[h][slot<K>(u, k + 1)][e];
                        dn[e] = sp[h][slot<K>(u, k - 1)][e];
                        nn[e] = sn[h][q][e];
                    } else {
                        cur[e] = w[h][s - 2][m][e];
                        up[e] = w[h][s - 2][slot<3>(u, k + 1)][e];
                        dn[e] = w[h][s - 2][slot<3>(u, k - 1)][e];
                        nn[e] = wn[h][s - 2][m][e];
                    }
                }
                // neighbours in x: the adjacent lanes' cells (and the lane's other one)
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
                    cell_rhs<R, RES>(c, cur[e], lr[e].x, lr[e].y, up[e].x + dn[e].x, up[e].y + dn[e].y, nn[e],
                                         sP[q][e], sk[q][e], fx, fy, fn);
                    if constexpr (DRIVE) {  // -(i/hbar) E ph
                        const C d = sE[q][e], p = ph[k - 1];
                        fx = fma(c.inv_hbar, d.x * p.y + d.y * p.x, fx);
                        fy = fma(-c.inv_hbar, d.x * p.x - d.y * p.y, fy);
                    }
                    C& ac = acc[h][a4][e];
                    R& an = accn[h][a4][e];
                    const C p0 = sp[h][q][e];
                    const R n0 = sn[h][q][e];
                    if (s < 4) {
                        const R step = s == 3 ? a.dt : a.half_dt;
                        ac = s == 1 ? C{fx, fy} : C{fma(R(2), fx, ac.x), fma(R(2), fy, ac.y)};
                        an = s == 1 ? fn : fma(R(2), fn, an);
                        w[h][s - 1][m][e] = C{kk * fma(step, fx, p0.x), kk * fma(step, fy, p0.y)};
                        wn[h][s - 1][m][e] = kk * fma(step, fn, n0);
                        keep_here(ac);
                        keep_here(w[h][s - 1][m][e]);
                        if (RES) {
                            keep_here(an);
                            keep_here(wn[h][s - 1][m][e]);
                        }
                    } else {
                        y[e] = C{fma(a.dt6, ac.x + fx, p0.x), fma(a.dt6, ac.y + fy, p0.y)};
                        yn[e] = fma(a.dt6, an + fn, n0);
                        if (h == 0) {  // the state in between (0 in ghost cells)
                            sp[1][q][e] = C{kk * y[e].x, kk * y[e].y};
                            sn[1][q][e] = kk * yn[e];
                            keep_here(sp[1][q][e]);
                            if (RES) keep_here(sn[1][q][e]);
                        }
                    }
                }
                if (k == 8) {
                    // issued at every position (no branch); a row outside the band goes to
                    // a descriptor of size 0, whose stores are dropped
                    const bool st = r >= b0 && r < b0 + B && r < a.ny;  // uniform
                    const int rr = st ? r : 0;
                    if constexpr (W == 2) {
                        wstore4(wf4{y[0].x, y[0].y, y[1].x, y[1].y}, st ? rpo : rnull, oc, rr * rowc);
                        if (RES) wstore2(wf2{yn[0], yn[1]}, st ? rno : rnull, orr, rr * rowr);
                    } else {
                        buf_store_nt(y[0], st ? rpo : rnull, (int)((unsigned)oc + (unsigned)(rr * rowc)));
                        if (RES) buf_store_nt(yn[0], st ? rno : rnull, (int)((unsigned)orr + (unsigned)(rr * rowr)));
                    }
                    if (CHECK) {
                        R t = nf;  // stays 0 while the stored values are finite
#pragma unroll
                        for (int e = 0; e < W; ++e) {
                            t = fma(y[e].x, R(0), t);
                            t = fma(y[e].y, R(0), t);
                            if (RES) t = fma(yn[e], R(0), t);
                        }
                        nf = st ? t : nf;
                    }
                }
            }
            if (W == 1 && sizeof(R) == 4 && !FIRST && (u == 3 || u == 7) && base + u + 1 >= npos) {  // uniform
                finish(CHECK && out_col && !(nf == R(0)));
                __builtin_amdgcn_endpgm();
            }
        }
    };
    positions(std::true_type{}, 0);
    // npos > K: the bands have at least 8 rows
    for (int base = K; base < npos; base += K) positions(std::false_type{}, base);
    finish(CHECK && out_col && !(nf == R(0)));
}

template <typename R, int W, bool RES, bool HASV, bool GHOSTS, bool YZERO, int WPE, bool CHECK, bool DRIVE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPE)))
void rk4_stream_pair_kernel(const StepArgs<R> a)
{
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const int band = t / a.tiles_x, strip = t - band * a.tiles_x;
    stream_band_pair<R, W, RES, HASV, GHOSTS, YZERO, CHECK, DRIVE>(a, strip, band, a.band_rows, (band & 1) ? -1 : 1,
                                                                [&](bool bad) __attribute__((always_inline)) {
                                                                    if (bad) a.flag[0] = 1u;  // benign race
                                                                });
}

}  // namespace phx
