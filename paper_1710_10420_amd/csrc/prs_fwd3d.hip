// prs_fwd3d.hip -- 3D multi-step passes, for the field precision
// PRS_REAL (float or double) this translation unit is compiled for; the
// device templates are in prs_device.h.  One unit per dimension, direction
// and precision, so that they compile in parallel.

#include "prs_device.h"

#ifndef PRS_REAL
#error "compile with -DPRS_REAL=float or -DPRS_REAL=double"
#endif

namespace prs {

template <typename R>
hipError_t launch_tb3d(int T, const Geometry& g, const Tiling& t, const void* phi_in, void* phi_out,
                       const void* pi_in, void* pi_out, const StepCoef64* k, bool diag, WavePartial* partials,
                       const DiagCoef& dc, int halo, hipStream_t s)
{
    return launch_tb3d_r<R>(T, g, t, phi_in, phi_out, pi_in, pi_out, k, diag, partials, dc, s, halo);
}

template hipError_t launch_tb3d<PRS_REAL>(int T, const Geometry& g, const Tiling& t, const void* phi_in,
                                          void* phi_out, const void* pi_in, void* pi_out, const StepCoef64* k,
                                          bool diag, WavePartial* partials, const DiagCoef& dc, int halo,
                                          hipStream_t s);

template <typename R>
hipError_t launch_tb3_deep_p(const Geometry& g, const Tiling& t, const void* phi_in, void* phi_out,
                             const void* pi_in, void* pi_out, const StepCoef64* k, hipStream_t s)
{
    constexpr int VEC = sizeof(R) == 4 ? 2 : 1;     // 512 bytes a wave and row
    if (t.vec != VEC || tb3l_waves(t.ty) != 8 || tb3l_rows_per_wave(t.ty) != 4) return hipErrorInvalidValue;
    return launch_tb3l_t<R, VEC, kDeepSteps, 4, 8, false>(g, t, phi_in, phi_out, pi_in, pi_out, nullptr, k, false, nullptr,
                                                   DiagCoef{}, s);
}

template hipError_t launch_tb3_deep_p<PRS_REAL>(const Geometry& g, const Tiling& t, const void* phi_in,
                                                void* phi_out, const void* pi_in, void* pi_out, const StepCoef64* k,
                                                hipStream_t s);

}  // namespace prs
