// Dispatch of the streaming whole-step RK4 kernel for the two-component (spinor) form
// (stream_spinor.h); its variants are instantiated in units of their own.
#include "stream_spinor_launch.h"

namespace phx {

extern template hipError_t launch_spinor_part<float, 2, false, false, false>(bool, const StepArgs<float>&, hipStream_t);
extern template hipError_t launch_spinor_part<float, 1, false, false, false>(bool, const StepArgs<float>&, hipStream_t);
extern template hipError_t launch_spinor_part<double, 1, false, false, false>(bool, const StepArgs<double>&, hipStream_t);
extern template hipError_t launch_spinor_part<float, 1, true, false, false>(bool, const StepArgs<float>&, hipStream_t);
extern template hipError_t launch_spinor_part<double, 1, true, false, false>(bool, const StepArgs<double>&, hipStream_t);
extern template hipError_t launch_spinor_part<float, 1, false, true, false>(bool, const StepArgs<float>&, hipStream_t);
extern template hipError_t launch_spinor_part<double, 1, false, true, false>(bool, const StepArgs<double>&, hipStream_t);
extern template hipError_t launch_spinor_part<float, 1, false, false, true>(bool, const StepArgs<float>&, hipStream_t);
extern template hipError_t launch_spinor_part<double, 1, false, false, true>(bool, const StepArgs<double>&, hipStream_t);

template <typename R>
hipError_t launch_stream_spinor(bool reservoir, bool has_v, const StepArgs<R>& a, hipStream_t s)
{
    if (a.imag_partials || a.E) {  // imaginary time, the coherent drive: without reservoirs
        if (reservoir) return hipErrorInvalidValue;
        return a.E ? launch_spinor_part<R, 1, false, false, true>(has_v, a, s)
                   : launch_spinor_part<R, 1, false, true, false>(has_v, a, s);
    }
    if (reservoir) return launch_spinor_part<R, 1, true, false, false>(has_v, a, s);
    if constexpr (sizeof(R) == 4) {
        if (a.columns == 2) return launch_spinor_part<R, 2, false, false, false>(has_v, a, s);
    }
    return launch_spinor_part<R, 1, false, false, false>(has_v, a, s);
}

template hipError_t launch_stream_spinor<float>(bool, bool, const StepArgs<float>&, hipStream_t);
template hipError_t launch_stream_spinor<double>(bool, bool, const StepArgs<double>&, hipStream_t);

// Columns per lane, strips and band height (a multiple of 8; `rows` where the caller gave
// one).  Two columns per lane need 16-byte rows (complex64, even width) and registers
// (no reservoirs, imaginary time or drive); they take fewer instructions per cell, one
// column gives more and shorter waves on grids that do not fill the device: 21.0 against
// 23.0 us per step at 1024^2, 12.0 against 13.5 at 512^2.
SpinorPlan spinor_plan(const phx_config& c, int rows, int cus)
{
    const bool c64 = c.precision == PHX_C64, res = c.reservoir != 0, imag = c.imag_time != 0, drive = c.drive != 0;
    SpinorPlan best{};
    double cost = 0.0;
    for (int w = 1; w <= (c64 && c.nx % 2 == 0 && !res && !imag && !drive ? 2 : 1); ++w) {
        const int strips = (c.nx + spinor_cols(w) - 1) / spinor_cols(w);
        const BandFill f = band_fill(strips, c.ny, 8, 5, 8, 8, cus, spinor_waves_per_simd(c64, w, res, imag, drive));
        const double t = f.cost * spinor_instructions(w);
        if (w == 1 || t < cost) {
            cost = t;
            best = SpinorPlan{w, strips, rows > 0 ? rows : f.rows};
        }
    }
    return best;
}

}  // namespace phx
