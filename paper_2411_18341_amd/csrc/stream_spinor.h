// Device code of the streaming whole-step RK4 kernel for the two-component (spinor)
// form of Eqs. (PULSE_psi), (PULSE_res): self and cross interaction, the potential,
// the TE-TM coupling J_+- = Delta_LT (d_x -+ i d_y)^2, whose mixed derivative needs
// the diagonal neighbours of the other component, and (RES) the reservoirs n_+-
// with gain, reservoir interaction and pumps P_+-.
//
// The band walk is the one-component kernel's (stream_step.h): one wave per strip of
// columns plus a 4-column halo (W = 1 column per lane: 56 output columns; W = 2, complex64
// without reservoirs on even widths: 120), rows walked once with the four stages pipelined
// one row apart, inputs in an 8-row ring, running sums and stage arguments in rings of 4 --
// here for both components.  x-neighbours come from DPP lane shifts; the mixed difference
//   X = o[i+1,j+1] - o[i+1,j-1] - o[i-1,j+1] + o[i-1,j-1]
// is the shift by one column of (row below - row above) of the other component, and
// changes sign with the walking direction (odd bands walk upwards).
//
// The kernel is bound by its VALU issue, so what counts is the number of instructions:
// two columns per lane halve the halo columns (128 / 120 instead of 64 / 56) and leave one
// lane shift per neighbour sum instead of two; bands are as tall as the device's wave
// slots allow, so that all waves run at once (with bands of 64 rows 4096^2 took one and a
// half rounds of waves); stage s starts at position 2 s, before which no stage needs its
// rows.  Every ring length divides the 8 positions of the unrolled body; the values that
// later positions read are pinned where they are formed (keep_here).  Measured, us per
// step with zero boundaries and a potential (before: one column per lane, bands of 40 rows,
// 24 positions unrolled): complex64 143 (186) at 4096^2, 49.7 (75.2) at 2048^2, 9.6 (34.2) at
// 512^2; with reservoirs 64.6 (96.4) at 2048^2; complex128 75.9 (108.7) at 2048^2; drive 61.2
// (102.2), imaginary time with its norm pass 56.4 (90.5) at 2048^2.  At 4096^2 the 2030 waves of
// 80 positions issue 532 VALU instructions each, 137 us back to back.
#pragma once

#include <type_traits>

#include "stream_wide.h"

namespace phx {

// f_s for both components from the stage arguments (cur), the neighbour sums in x
// (lr) and y (ud), the y-differences of the rows below and above (dy = below - above,
// for the mixed term), the per-cell constant kv = V/hbar + 2 (ax + ay) and (RES) the
// reservoir values nn and pumps pv.
//   f_s = i T_s + (u_s - i om_s) p_s - sgn_s bxy X_o,   u_s = (R n_s - gamma)/2,
//   T_s = ax lr_s + ay ud_s - 2(ax + ay) p_s - bx (lr_o - 2 q) + by (ud_o - 2 q),
//   om_s = V/hbar + gh rho_s + gxh rho_o + grh n_s (the -2(ax + ay) p_s term folded into kv),
//   fn_s = P_s - (gamma_r + R rho_s) n_s,
// X_o = dir (next(dy_o) - prev(dy_o)), sgn = +1 for psi_+, -1 for psi_-; dir bxy is passed in as
// bxyd (dir is +-1: the same value bit for bit as multiplying X by dir).
template <typename R, bool RES, bool IMAG = false>
__device__ __forceinline__ void spinor_rhs(const Coef<R>& c, const typename cvec<R>::type (&cur)[2],
                                           const typename cvec<R>::type (&lr)[2],
                                           const typename cvec<R>::type (&ud)[2],
                                           const typename cvec<R>::type (&xx)[2], R kv, R bxyd,
                                           const R (&nn)[2], const R (&pv)[2], typename cvec<R>::type (&f)[2],
                                           R (&fn)[2])
{
    using C = typename cvec<R>::type;
    const R rho0 = fma(cur[0].x, cur[0].x, cur[0].y * cur[0].y);
    const R rho1 = fma(cur[1].x, cur[1].x, cur[1].y * cur[1].y);
    const R cb = R(2) * (c.bx - c.by);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int o = 1 - s;
        const C p = cur[s], q = cur[o];
        const R rs = s == 0 ? rho0 : rho1;
        R om = fma(c.gh, rs, fma(c.gxh, s == 0 ? rho1 : rho0, kv));
        if (RES) om = fma(c.grh, nn[s], om);
        const R u = RES ? fma(c.half_R, nn[s], -c.half_gamma) : -c.half_gamma;
        fn[s] = RES ? fma(-fma(c.R_, rs, c.gamma_r), nn[s], pv[s]) : R(0);
        // other component's second differences: -bx (lr_o - 2q) + by (ud_o - 2q)
        const R ox = fma(-c.bx, lr[o].x, fma(c.by, ud[o].x, cb * q.x));
        const R oy = fma(-c.bx, lr[o].y, fma(c.by, ud[o].y, cb * q.y));
        const R tx = fma(c.ax, lr[s].x, fma(c.ay, ud[s].x, ox));
        const R ty = fma(c.ax, lr[s].y, fma(c.ay, ud[s].y, oy));
        // the walking direction's sign rides on the coefficient (bxyd = dir bxy, chosen
        // once per band), not on each difference
        const R sb = s == 0 ? -bxyd : bxyd;
        f[s].x = fma(sb, xx[o].x, fma(u, p.x, fma(om, p.y, -ty)));
        f[s].y = fma(sb, xx[o].y, fma(u, p.y, fma(-om, p.x, tx)));
        if constexpr (IMAG) {  // imaginary time: -i f
            const R t = f[s].x;
            f[s].x = f[s].y;
            f[s].y = -t;
        }
    }
}

constexpr int spinor_cols(int w) { return 64 * w - 8; }  // output columns per strip

// Waves per SIMD that the registers allow without scratch memory.
constexpr int spinor_waves_per_simd(bool c64, int w, bool res, bool imag, bool drive)
{
    if (!c64) return res || drive ? 1 : 2;
    if (w == 2 || res) return 2;
    return imag || drive ? 3 : 4;
}
// VALU instructions of one position (four stages, one row of the lane's columns).
constexpr int spinor_instructions(int w) { return w == 2 ? 532 : 297; }

// One band of `B` rows (a multiple of 8) of strip `strip`; `finish(bad, norm)` gets whether
// a stored value is not finite and the lane's norm partial.
// IMAG: imaginary time (no reservoirs): each stage's derivative is rotated by -i, the
// input is multiplied by the scale that restores the previous step's
// norm, and the norm partial is this lane's FP64 sum of |psi_out|^2 over both components
// of the cells it stores.
// DRIVE (no reservoirs, real time): the coherent drive -(i/hbar) E_s(r) exp(-i omega t_k)
// joins the derivative of component s at stage k; both components of E ride in the
// input ring beside psi, the four stage phasors come from a.drive_ph.
template <typename R, int W, bool RES, bool HASV, bool GHOSTS, bool YZERO, bool IMAG, bool DRIVE, typename F>
__device__ __forceinline__ void stream_band_spinor(const StepArgs<R>& a, int strip, int band, int B, int dir, F finish)
{
    static_assert(!(IMAG && RES), "imaginary time has no reservoir");
    static_assert(!(DRIVE && (RES || IMAG)), "the drive runs without reservoirs, in real time");
    static_assert(W == 1 || (W == 2 && sizeof(R) == 4 && !RES && !IMAG && !DRIVE), "two columns per lane: complex64");
    using C = typename cvec<R>::type;
    constexpr int K = 8;              // rows j - 4 .. j + PF are in flight
    // rows loaded ahead of their first use
    constexpr int PF = W == 2 ? 2 : 3;
    const R sc = IMAG ? imag_scale(a) : R(1);  // uniform
    double nrm = 0.0;
    const int lane = threadIdx.x & 63;
    const Coef<R>& c = a.c;
    const int gi = strip * spinor_cols(W) - 4 + W * lane;
    const int ci = wrap_any(gi, a.nx, a.bcx);
    const bool gcol = GHOSTS && ci < 0;
    // Ghost columns and rows stay 0 in every stage: their inputs read as 0, so the stage
    // argument p0 + h f is 0 there when the step h is taken as 0 (the lane's h values,
    // and per row a uniform choice between them and 0).
    R kh2 = gcol ? R(0) : a.half_dt;
    R kh = gcol ? R(0) : a.dt;
    const int b0 = band * B;
    const R kdiag = R(2) * (c.ax + c.ay);
    const R bxyd = dir > 0 ? c.bxy : -c.bxy;  // uniform over the wave
    const size_t cells = (size_t)a.nx * a.ny;
    const __amdgpu_buffer_rsrc_t rpo = buffer_of(a.psi_out, 2 * cells * sizeof(C));
    const __amdgpu_buffer_rsrc_t rno = buffer_of(a.n_out, RES ? 2 * cells * sizeof(R) : 0);
    // inputs through buffer loads: the lane's column offset in a VGPR (past the buffer
    // for a ghost column, which then reads 0), the row and component offsets in
    // scalars; a ghost row (zero y boundary) reads through a descriptor of size 0
    const __amdgpu_buffer_rsrc_t rpi = buffer_of(a.psi_in, 2 * cells * sizeof(C));
    const __amdgpu_buffer_rsrc_t rni = buffer_of(a.n_in, RES ? 2 * cells * sizeof(R) : 0);
    const __amdgpu_buffer_rsrc_t rP = buffer_of(a.P, RES ? 2 * cells * sizeof(R) : 0);
    const __amdgpu_buffer_rsrc_t rV = buffer_of(a.V, HASV ? cells * sizeof(R) : 0);
    const __amdgpu_buffer_rsrc_t rnull = buffer_of(a.psi_in, 0);
    const __amdgpu_buffer_rsrc_t rE = buffer_of(a.E, DRIVE ? 2 * cells * sizeof(C) : 0);

    // [component][slot][column of the lane]
    C sp[2][K][W], sE[2][K][W];  // state; DRIVE: the profile
    R sk[K][W];
    R sn[2][K][W], sP[2][K][W];
    C acc[2][4][W], w[2][3][4][W];  // w[.][q]: argument of stage q + 2
    R accn[2][4][W], wn[2][3][4][W];
#pragma unroll
    for (int e = 0; e < W; ++e)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
#pragma unroll
            for (int s = 0; s < K; ++s) {
                sp[m][s][e] = sE[m][s][e] = czero<C>();
                sn[m][s][e] = sP[m][s][e] = R(0);
                sk[s][e] = kdiag;
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                acc[m][s][e] = czero<C>();
                accn[m][s][e] = R(0);
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    w[m][q][s][e] = czero<C>();
                    wn[m][q][s][e] = R(0);
                }
            }
        }
    C ph[4];  // DRIVE: the phasors of the four stage times
    if constexpr (DRIVE) {
#pragma unroll
        for (int s = 0; s < 4; ++s) ph[s] = a.drive_ph[s];
    }
    // DRIVE: adds -(i/hbar) E ph to f
    auto drive = [&](C& f, const C e, const C p) {
        const R zx = e.x * p.x - e.y * p.y;
        const R zy = e.x * p.y + e.y * p.x;
        f.x = fma(c.inv_hbar, zy, f.x);
        f.y = fma(-c.inv_hbar, zx, f.y);
    };

    const int npos = B + 8;
    const int start = dir > 0 ? b0 - 4 : b0 + B + 3;
    int g = start;
    int rw = wrap_any(g, a.ny, a.bcy);
    const int ci0 = ci < 0 ? 0 : ci;
    const int vc = gcol ? kOutOfRange : ci0 * (int)sizeof(C);
    const int vr = gcol ? kOutOfRange : ci0 * (int)sizeof(R);
    const int comp_c = (int)(cells * sizeof(C)), comp_r = (int)(cells * sizeof(R));
    const int row_c = a.nx * (int)sizeof(C), row_r = a.nx * (int)sizeof(R);
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
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            load_c(grow ? rnull : rpi, sp[m][s], m * comp_c + rr * row_c);
            if constexpr (DRIVE) load_c(grow ? rnull : rE, sE[m][s], m * comp_c + rr * row_c);
            if (RES) {
                load_r(grow ? rnull : rni, sn[m][s], m * comp_r + rr * row_r);
                load_r(grow ? rnull : rP, sP[m][s], m * comp_r + rr * row_r);
            }
        }
        if (HASV) load_r(grow ? rnull : rV, sk[s], rr * row_r);
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
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                if constexpr (IMAG) sp[m][q][e] = C{sp[m][q][e].x * sc, sp[m][q][e].y * sc};
                keep_here(sp[m][q][e]);
                if constexpr (DRIVE) keep_here(sE[m][q][e]);
                if (RES) {
                    keep_here(sn[m][q][e]);
                    keep_here(sP[m][q][e]);
                }
            }
            if (HASV) {
                sk[q][e] = fma(c.inv_hbar, sk[q][e], kdiag);
                keep_here(sk[q][e]);
            }
        }
    };
#pragma unroll
    for (int t = 0; t < PF; ++t) fetch(t, true);

    // the lane's step h, or 0 on a ghost row (zero y boundary; uniform over the wave)
    auto row_h = [&](int r, R h) { return (YZERO && (unsigned)r >= (unsigned)a.ny) ? R(0) : h; };

    R nf = R(0);  // not 0: a value was not finite
    const bool out_col = lane >= 4 / W && lane < 64 - 4 / W && gi < a.nx;
    auto positions = [&](auto phase, int base) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(phase)::value;
#pragma unroll
        for (int u = 0; u < K; ++u) {
            const int j = start + dir * (base + u);
            fetch(slot<K>(u, -PF), base + u + PF < npos);
            arrive(slot<K>(u, 0));
            if constexpr (sizeof(R) == 8 && RES) {
                park(kh);
                park(kh2);
            }
#pragma unroll
            for (int s = 1; s <= 4; ++s) {
                if (FIRST && u < 2 * s) continue;
                const int q = slot<K>(u, s), m4 = slot<4>(u, s);
                const int r = j - s * dir;
                __builtin_amdgcn_sched_barrier(0);
                C lr[2][W], ud[2][W], dy[2][W], cur[2][W];
#pragma unroll
                for (int m = 0; m < 2; ++m) {
#pragma unroll
                    for (int e = 0; e < W; ++e) {
                        cur[m][e] = s == 1 ? sp[m][q][e] : w[m][s - 2][m4][e];
                        const C up = s == 1 ? sp[m][slot<K>(u, 2)][e] : w[m][s - 2][slot<4>(u, s + 1)][e];
                        const C dn = s == 1 ? sp[m][slot<K>(u, 0)][e] : w[m][s - 2][slot<4>(u, s - 1)][e];
                        ud[m][e] = C{up.x + dn.x, up.y + dn.y};
                        dy[m][e] = C{dn.x - up.x, dn.y - up.y};
                    }
                    if constexpr (W == 2) {
                        lr[m][0] = C{lane_prev(cur[m][1].x) + cur[m][1].x, lane_prev(cur[m][1].y) + cur[m][1].y};
                        lr[m][1] = C{cur[m][0].x + lane_next(cur[m][0].x), cur[m][0].y + lane_next(cur[m][0].y)};
                    } else {
                        lr[m][0] = C{lane_prev(cur[m][0].x) + lane_next(cur[m][0].x),
                                     lane_prev(cur[m][0].y) + lane_next(cur[m][0].y)};
                    }
                }
                const R hk = row_h(r, s == 3 ? kh : kh2);
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    // the mixed difference of each component: right minus left column
                    C xx[2], f[2];
                    R fn[2], nn[2], pv[2];
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        if constexpr (W == 2)
                            xx[m] = e == 0 ? C{dy[m][1].x - lane_prev(dy[m][1].x), dy[m][1].y - lane_prev(dy[m][1].y)}
                                           : C{lane_next(dy[m][0].x) - dy[m][0].x, lane_next(dy[m][0].y) - dy[m][0].y};
                        else
                            xx[m] = C{lane_next(dy[m][0].x) - lane_prev(dy[m][0].x),
                                      lane_next(dy[m][0].y) - lane_prev(dy[m][0].y)};
                        nn[m] = s == 1 ? sn[m][q][e] : wn[m][s - 2][m4][e];
                        pv[m] = sP[m][q][e];
                    }
                    const C cu[2] = {cur[0][e], cur[1][e]}, l2[2] = {lr[0][e], lr[1][e]}, u2[2] = {ud[0][e], ud[1][e]};
                    spinor_rhs<R, RES, IMAG>(c, cu, l2, u2, xx, sk[q][e], bxyd, nn, pv, f, fn);
                    if constexpr (DRIVE) {
                        drive(f[0], sE[0][q][e], ph[s - 1]);
                        drive(f[1], sE[1][q][e], ph[s - 1]);
                    }
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        C& ac = acc[m][m4][e];
                        R& an = accn[m][m4][e];
                        const C p0 = sp[m][q][e];
                        const R n0 = sn[m][q][e];
                        if (s < 4) {
                            ac = s == 1 ? f[m] : C{fma(R(2), f[m].x, ac.x), fma(R(2), f[m].y, ac.y)};
                            w[m][s - 1][m4][e] = C{fma(hk, f[m].x, p0.x), fma(hk, f[m].y, p0.y)};
                            keep_here(ac);
                            keep_here(w[m][s - 1][m4][e]);
                            if (RES) {
                                an = s == 1 ? fn[m] : fma(R(2), fn[m], an);
                                wn[m][s - 1][m4][e] = fma(hk, fn[m], n0);
                                keep_here(an);
                                keep_here(wn[m][s - 1][m4][e]);
                            }
                        } else {
                            // the finished row (kept in the dead sums until both columns are done)
                            ac = C{fma(a.dt6, ac.x + f[m].x, p0.x), fma(a.dt6, ac.y + f[m].y, p0.y)};
                            if (RES) an = fma(a.dt6, an + fn[m], n0);
                        }
                    }
                }
                if (s == 4) {
                    // stored when it lies in the band and in the grid (else the store goes to
                    // the empty descriptor or an out-of-range column and is dropped)
                    const bool st = r >= b0 && r < b0 + B && r < a.ny;  // uniform
                    const int rr = st ? r : 0;
                    R t = nf;
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        const int oc = out_col ? gi * (int)sizeof(C) : kOutOfRange;
                        const int orr = out_col ? gi * (int)sizeof(R) : kOutOfRange;
                        const C* y = acc[m][m4];
                        const unsigned off = (unsigned)oc + (unsigned)(m * comp_c + rr * row_c);
                        if constexpr (W == 2)
                            wstore4(wf4{y[0].x, y[0].y, y[1].x, y[1].y}, st ? rpo : rnull, (int)off, 0);
                        else
                            buf_store_nt(y[0], st ? rpo : rnull, (int)off);
                        if constexpr (RES)
                            buf_store_nt(accn[m][m4][0], st ? rno : rnull,
                                         (int)((unsigned)orr + (unsigned)(m * comp_r + rr * row_r)));
#pragma unroll
                        for (int e = 0; e < W; ++e) {
                            if constexpr (IMAG)
                                nrm += st && out_col ? (double)y[e].x * y[e].x + (double)y[e].y * y[e].y : 0.0;
                            t = fma(y[e].x, R(0), t);  // stays 0 while the values are finite
                            t = fma(y[e].y, R(0), t);
                            if (RES) t = fma(accn[m][m4][e], R(0), t);
                        }
                    }
                    nf = st ? t : nf;
                }
            }
        }
    };
    positions(std::true_type{}, 0);
    for (int base = K; base < npos; base += K) positions(std::false_type{}, base);
    finish(out_col && !(nf == R(0)), nrm);
}

}  // namespace phx
