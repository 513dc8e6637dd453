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

}  // namespace prs
