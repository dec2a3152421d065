// Whole-attempt Dormand-Prince kernel: the seven stages of RK5(4)7M, the fifth-order
// solution and the embedded error of one attempted step in one pass over the state.
//
// One wave per strip of columns walks a band of rows, as the streaming RK4 step does
// (stream_step.h): at row j stage s runs at row j - s, so the rows that a stage needs
// (r - 1, r, r + 1 of its argument) were finished by the stage before it at this or an
// earlier row.  K_1..K_6 of the rows in flight stay in registers until the error of
// their row is formed, so neither K_s nor a stage argument goes through memory: an
// attempt reads psi (with n, P, V) and writes the new state, 36 bytes per point for
// the complex64 spinor with a potential instead of the 568 of one launch per stage.
// Seven stencils in a row make the halo 7 cells on each side (64 lanes give 50 output
// columns) and the walk B + 14 rows for B output rows; K_1 is evaluated again rather
// than read from the attempt before (the same value bit for bit, from the same state).
//
// The kernel is bound by its VALU issue: about 800 instructions per position of the
// complex64 spinor, i.e. 490 us at 4096^2 if they issue back to back, 513 us measured
// per attempt with the error sum and the host's turn (2595 us with one launch per
// stage, which is bound by HBM; complex128 driven 2048^2 150 against 996 us, complex64
// trap 512^2 29 against 53 us).  Rings are indexed by the row modulo 9 (rows j - 7 ..
// j + 1 are in flight) and the walk is unrolled by 9, so every slot is a fixed
// register.  One row of loads ahead of its use is enough here: a position takes
// thousands of cycles.  The wave ends inside the unrolled positions (s_endpgm): an exit
// that left the loop would make every ring slot live to a common end (237 instead of
// more than 305 registers for the complex64 spinor).
#pragma once

#include "stream_body.h"

namespace phx {

// Arguments of one attempt (the coefficients already contain dt).
template <typename R>
struct DpWalkArgs {
    using C = typename cvec<R>::type;
    int nx, ny, bcx, bcy;
    int strips, band_rows, tiles;
    Coef<R> c;
    const C* psi; const R* n;     // state at the start of the attempt
    const R* V;  const R* P;
    C* psi_out; R* n_out;         // fifth-order solution
    R ca[6][6];                   // ca[s-1][j-1] = dt a_{s+1,j}
    R ce[7];                      // dt (b_j - bhat_j)
    double rtol, atol;
    double* partials;             // one error partial per wave
};

// Waves per SIMD that the registers of a variant allow without scratch memory: the K_s
// and rings in flight take up to 168 VGPRs in complex64 (about 200 with the reservoir and a
// potential), 240 for the spinor, more than 256 (one wave) with its reservoirs; twice
// as many in complex128.  The variant that leaves stages out (skip) needs a few more.
constexpr int dp_waves_per_simd(bool c64, int comps, bool res, bool hasv, bool skip)
{
    if (c64) return comps == 1 ? (res && (hasv || skip) ? 2 : 3) : (res ? 1 : 2);
    return comps == 1 && !res ? 2 : 1;
}

constexpr int kDpSkipRows = 64;  // bands below this height leave out the stages no output needs
// lanes 7 .. 56 of a strip hold its output columns
constexpr int kDpHalo = 7, kDpCols = 64 - 2 * kDpHalo;

// Right-hand side of one cell in the operation order of rhs_cell (stencil.h) as the
// stage kernels execute it, written with explicit fused operations so that both paths
// take the same steps: lr / ud are the sums of the x and y neighbours, xx the mixed
// difference of each component, sbxy = dir * bxy, `second` marks stage 2 (whose two-component
// form adds the interaction with the reservoir in the other order).
template <typename R, int COMPS, bool RES, bool HASV>
__device__ __forceinline__ void dp_rhs(const Coef<R>& k, const typename cvec<R>::type (&p)[COMPS],
                                       const typename cvec<R>::type (&lr)[COMPS],
                                       const typename cvec<R>::type (&ud)[COMPS],
                                       const typename cvec<R>::type (&xx)[COMPS], R sbxy, const R (&nn)[COMPS], R v,
                                       bool second, typename cvec<R>::type (&f)[COMPS], R (&rho)[COMPS])
{
    using C = typename cvec<R>::type;
    C sx[COMPS], sy[COMPS];
#pragma unroll
    for (int s = 0; s < COMPS; ++s) {
        rho[s] = COMPS == 2 ? fma(p[s].x, p[s].x, p[s].y * p[s].y) : fma(p[s].y, p[s].y, p[s].x * p[s].x);
        sx[s] = C{fma(R(-2), p[s].x, lr[s].x), fma(R(-2), p[s].y, lr[s].y)};
        sy[s] = C{fma(R(-2), p[s].x, ud[s].x), fma(R(-2), p[s].y, ud[s].y)};
    }
#pragma unroll
    for (int s = 0; s < COMPS; ++s) {
        const int o = COMPS - 1 - s;
        R tx = fma(k.ax, sx[s].x, k.ay * sy[s].x);
        R ty = fma(k.ax, sx[s].y, k.ay * sy[s].y);
        R om = k.gh * rho[s];
        if (RES) om = COMPS == 2 && second ? fma(k.grh, nn[s], om) : fma(k.gh, rho[s], k.grh * nn[s]);
        if (HASV) om = fma(k.inv_hbar, v, om);
        const R u = RES ? fma(nn[s], k.half_R, -k.half_gamma) : -k.half_gamma;
        if constexpr (COMPS == 2) {
            tx += fma(k.by, sy[o].x, -(k.bx * sx[o].x));
            ty += fma(k.by, sy[o].y, -(k.bx * sx[o].y));
            om = fma(k.gxh, rho[o], om);
            const R sb = s == 0 ? -sbxy : sbxy;
            f[s].x = fma(om, p[s].y, fma(u, p[s].x, fma(sb, xx[o].x, -ty)));
            f[s].y = fma(-om, p[s].x, fma(u, p[s].y, fma(sb, xx[o].y, tx)));
        } else {
            f[s].x = fma(om, p[s].y, u * p[s].x) - ty;
            f[s].y = fma(u, p[s].y, -(om * p[s].x)) + tx;
        }
    }
}

// A value that is not used: any register will do.
__device__ __forceinline__ float any_value(float v) { return __builtin_nondeterministic_value(v); }
__device__ __forceinline__ double any_value(double v) { return __builtin_nondeterministic_value(v); }
template <typename C>
__device__ __forceinline__ C any_value(const C& v)
{
    return C{any_value(v.x), any_value(v.y)};
}

// One band of a.band_rows rows of strip `strip`; hands this lane's sum of the weighted
// squared errors of the cells it owns to `finish` and ends the wave.  GHOSTS: some
// boundary is zero; the stage arguments of cells outside the grid are then held at 0.
// SKIP: stage s is left out at the first 2 s positions, whose rows no output needs.
template <typename R, int COMPS, bool RES, bool HASV, bool GHOSTS, bool SKIP, typename F>
__device__ __forceinline__ void dp_band(const DpWalkArgs<R>& a, int strip, int band, int dir, F finish)
{
    using C = typename cvec<R>::type;
    constexpr int K = 9;
    // the next position's row is loaded before this stage: late where two waves share the
    // register file, so that its registers are taken for a shorter time
    constexpr int kFetchStage = sizeof(R) == 8 && RES ? 1 : 4;
    const int lane = threadIdx.x & 63;
    const int B = a.band_rows;
    const int gi = strip * kDpCols - kDpHalo + lane;
    const int ci = wrap_any(gi, a.nx, a.bcx);
    const bool gcol = GHOSTS && ci < 0;
    const bool yzero = GHOSTS && a.bcy == PHX_BC_ZERO;  // uniform
    const int b0 = band * B;
    const R sbxy = dir > 0 ? a.c.bxy : -a.c.bxy;  // the mixed difference changes sign with the direction
    const size_t cells = (size_t)a.nx * a.ny;
    const __amdgpu_buffer_rsrc_t rpi = buffer_of(a.psi, COMPS * cells * sizeof(C));
    const __amdgpu_buffer_rsrc_t rni = buffer_of(a.n, RES ? COMPS * cells * sizeof(R) : 0);
    const __amdgpu_buffer_rsrc_t rP = buffer_of(a.P, RES ? COMPS * cells * sizeof(R) : 0);
    const __amdgpu_buffer_rsrc_t rV = buffer_of(a.V, HASV ? cells * sizeof(R) : 0);
    const __amdgpu_buffer_rsrc_t rpo = buffer_of(a.psi_out, COMPS * cells * sizeof(C));
    const __amdgpu_buffer_rsrc_t rno = buffer_of(a.n_out, RES ? COMPS * cells * sizeof(R) : 0);
    const __amdgpu_buffer_rsrc_t rnull = buffer_of(a.psi, 0);
    const int ci0 = ci < 0 ? 0 : ci;
    const int vc = gcol ? kOutOfRange : ci0 * (int)sizeof(C);
    const int vr = gcol ? kOutOfRange : ci0 * (int)sizeof(R);
    const int row_c = a.nx * (int)sizeof(C), row_r = a.nx * (int)sizeof(R);
    const int comp_c = (int)(cells * sizeof(C)), comp_r = (int)(cells * sizeof(R));
    const bool out_col = lane >= kDpHalo && lane < kDpHalo + kDpCols && gi < a.nx;

    C sp[COMPS][K];              // state
    R sn[COMPS][K], sP[COMPS][K], sV[K];
    C k[COMPS][6][K];            // K_1..K_6 of the rows in flight
    R kn[COMPS][6][K];
    C w[COMPS][8][3];            // w[.][s]: argument of stage s = 2..7, rows modulo 3
    R wn[COMPS][8][3];
#pragma unroll
    for (int m = 0; m < COMPS; ++m) {
#pragma unroll
        for (int s = 0; s < K; ++s) {
            sp[m][s] = czero<C>();
            sn[m][s] = sP[m][s] = R(0);
            sV[s] = R(0);
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                k[m][q][s] = czero<C>();
                kn[m][q][s] = R(0);
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                w[m][q][s] = czero<C>();
                wn[m][q][s] = R(0);
            }
    }

    const int npos = B + 2 * kDpHalo;
    const int start = dir > 0 ? b0 - kDpHalo : b0 + B - 1 + kDpHalo;
    int g = start;
    int rw = wrap_any(g, a.ny, a.bcy);
    // past the last row of the walk (use == false) the load repeats a row and is not used
    auto fetch = [&](int s, bool use) {
        const bool grow = yzero && rw < 0;  // uniform
        const int rr = grow ? 0 : rw;
#pragma unroll
        for (int m = 0; m < COMPS; ++m) {
            sp[m][s] = buf_load<C>(grow ? rnull : rpi, vc, m * comp_c + rr * row_c);
            if (RES) {
                sn[m][s] = buf_load<R>(grow ? rnull : rni, vr, m * comp_r + rr * row_r);
                sP[m][s] = buf_load<R>(grow ? rnull : rP, vr, m * comp_r + rr * row_r);
            }
        }
        if (HASV) sV[s] = buf_load<R>(grow ? rnull : rV, vr, rr * row_r);
        const int gn = g + dir;
        int rn;
        if (yzero) {
            rn = (gn >= 0 && gn < a.ny) ? gn : -1;
        } else {
            rn = rw + dir;
            rn = rn == a.ny ? 0 : (rn < 0 ? a.ny - 1 : rn);
        }
        g = use ? gn : g;
        rw = use ? rn : rw;
    };
    fetch(slot<K>(0, 0), true);

    double err = 0.0;
    for (int base = 0;; base += K) {
#pragma unroll
        for (int u = 0; u < K; ++u) {
            const int j = start + dir * (base + u);
            if (base + u >= npos) {  // uniform
                finish(err);
                __builtin_amdgcn_endpgm();
            }
#pragma unroll
            for (int s = 1; s <= 7; ++s) {
                const int q = slot<K>(u, s);  // ring slot of row r = j - s
                const int r = j - s * dir;
                if (s == kFetchStage) fetch(slot<K>(u, -1), base + u + 1 < npos);
                if (SKIP && base + u < 2 * s) {  // uniform: no later stage needs this row of stage s
                    if (s < 7) {
#pragma unroll
                        for (int m = 0; m < COMPS; ++m) {
                            w[m][s + 1][slot<3>(u, s)] = any_value(w[m][s + 1][slot<3>(u, s)]);
                            k[m][s - 1][q] = any_value(k[m][s - 1][q]);
                            if (RES) {
                                wn[m][s + 1][slot<3>(u, s)] = any_value(wn[m][s + 1][slot<3>(u, s)]);
                                kn[m][s - 1][q] = any_value(kn[m][s - 1][q]);
                            }
                        }
                    }
                    continue;
                }
                C cur[COMPS], lr[COMPS], ud[COMPS], xx[COMPS], f[COMPS];
                R nn[COMPS], rho[COMPS], fn[COMPS];
#pragma unroll
                for (int m = 0; m < COMPS; ++m) {
                    C up, dn;
                    if (s == 1) {
                        cur[m] = sp[m][q];
                        up = sp[m][slot<K>(u, 2)];
                        dn = sp[m][slot<K>(u, 0)];
                        nn[m] = sn[m][q];
                    } else {
                        cur[m] = w[m][s][slot<3>(u, s)];
                        up = w[m][s][slot<3>(u, s + 1)];
                        dn = w[m][s][slot<3>(u, s - 1)];
                        nn[m] = wn[m][s][slot<3>(u, s)];
                    }
                    lr[m] = C{lane_prev(cur[m].x) + lane_next(cur[m].x), lane_prev(cur[m].y) + lane_next(cur[m].y)};
                    ud[m] = C{up.x + dn.x, up.y + dn.y};
                    xx[m] = czero<C>();
                    if (COMPS == 2) {
                        const R dx = dn.x - up.x, dy = dn.y - up.y;
                        xx[m] = C{lane_next(dx) - lane_prev(dx), lane_next(dy) - lane_prev(dy)};
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                dp_rhs<R, COMPS, RES, HASV>(a.c, cur, lr, ud, xx, sbxy, nn, sV[q], s == 2, f, rho);
                const bool ghost = GHOSTS && (gcol || (yzero && (unsigned)r >= (unsigned)a.ny));
#pragma unroll
                for (int m = 0; m < COMPS; ++m) {
                    fn[m] = RES ? fma(-nn[m], fma(a.c.R_, rho[m], a.c.gamma_r), sP[m][q]) : R(0);
                    if (s < 7) {
                        // y_{s+1} = psi + sum_j dt a_{s+1,j} K_j, j in increasing order
                        C y = sp[m][q];
                        R yn = sn[m][q];
#pragma unroll
                        for (int jj = 0; jj < s - 1; ++jj) {
                            if (s == 6 && jj == 1) continue;  // a_72 = 0
                            y.x = fma(a.ca[s - 1][jj], k[m][jj][q].x, y.x);
                            y.y = fma(a.ca[s - 1][jj], k[m][jj][q].y, y.y);
                            if (RES) yn = fma(a.ca[s - 1][jj], kn[m][jj][q], yn);
                        }
                        y.x = fma(a.ca[s - 1][s - 1], f[m].x, y.x);
                        y.y = fma(a.ca[s - 1][s - 1], f[m].y, y.y);
                        if (GHOSTS) {
                            y.x = ghost ? R(0) : y.x;
                            y.y = ghost ? R(0) : y.y;
                        }
                        w[m][s + 1][slot<3>(u, s)] = y;
                        if (RES) {
                            yn = fma(a.ca[s - 1][s - 1], fn[m], yn);
                            wn[m][s + 1][slot<3>(u, s)] = yn;
                            kn[m][s - 1][q] = fn[m];
                        }
                        k[m][s - 1][q] = f[m];
                        if (s == 6) {  // y_7 is the fifth-order solution
                            const bool st = out_col && r >= b0 && r < b0 + B && r < a.ny;
                            const int cell = r * a.nx + gi;
                            buf_store_nt(y, rpo, st ? m * comp_c + cell * (int)sizeof(C) : kOutOfRange);
                            if (RES) buf_store_nt(yn, rno, st ? m * comp_r + cell * (int)sizeof(R) : kOutOfRange);
                        }
                    } else {
                        // embedded error e = sum_j dt (b_j - bhat_j) K_j  (b_2 = bhat_2 = 0)
                        const bool st = out_col && r >= b0 && r < b0 + B && r < a.ny;
                        C e = C{fma(a.ce[6], f[m].x, a.ce[0] * k[m][0][q].x),
                                fma(a.ce[6], f[m].y, a.ce[0] * k[m][0][q].y)};
                        R en = RES ? fma(a.ce[6], fn[m], a.ce[0] * kn[m][0][q]) : R(0);
#pragma unroll
                        for (int jj = 2; jj < 6; ++jj) {
                            e.x = fma(a.ce[jj], k[m][jj][q].x, e.x);
                            e.y = fma(a.ce[jj], k[m][jj][q].y, e.y);
                            if (RES) en = fma(a.ce[jj], kn[m][jj][q], en);
                        }
                        const C p0 = sp[m][q], p1 = cur[m];
                        const double m0 = (double)p0.x * p0.x + (double)p0.y * p0.y;
                        const double m1 = (double)p1.x * p1.x + (double)p1.y * p1.y;
                        // the square root is monotonic and correctly rounded: one of the larger modulus
                        const double sc = a.atol + a.rtol * sqrt(fmax(m0, m1));
                        double add = ((double)e.x * e.x + (double)e.y * e.y) / (sc * sc);
                        err += st ? add : 0.0;
                        if (RES) {
                            const double sq = a.atol + a.rtol * fmax(fabs((double)sn[m][q]), fabs((double)nn[m]));
                            add = (double)en * en / (sq * sq);
                            err += st ? add : 0.0;
                        }
                    }
                }
            }
        }
    }
}

template <typename R, int COMPS, bool RES, bool HASV, bool GHOSTS, bool SKIP, int WPE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPE)))
void dp_stream_kernel(const DpWalkArgs<R> a)
{
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const int band = t / a.strips, strip = t - band * a.strips;
    dp_band<R, COMPS, RES, HASV, GHOSTS, SKIP>(a, strip, band, (band & 1) ? -1 : 1, [&](double err) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) err += __shfl_xor(err, m, 64);
        if (threadIdx.x == 0) a.partials[t] = err;
    });
}

}  // namespace phx
