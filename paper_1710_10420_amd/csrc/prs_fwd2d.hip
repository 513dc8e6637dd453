// prs_fwd2d.hip -- 2D multi-step and block passes, for the field precision
// PRS_REAL (float or double) this translation unit is compiled for; the
// device templates are in prs_device.h.  One unit per dimension, direction
// and precision, so that they compile in parallel.

#include "prs_block2d.h"

#ifndef PRS_REAL
#error "compile with -DPRS_REAL=float or -DPRS_REAL=double"
#endif

namespace prs {

template <typename R>
hipError_t launch_tb2d(int T, const Geometry& g, const Tiling& t, const void* phi_in, void* phi_out,
                       const void* pi_in, void* pi_out, const StepCoef64* k, bool diag, WavePartial* partials,
                       const DiagCoef& dc, int halo, hipStream_t s)
{
    return launch_tb2d_r<R>(T, g, t, phi_in, phi_out, pi_in, pi_out, k, diag, partials, dc, s, halo);
}

template hipError_t launch_tb2d<PRS_REAL>(int T, const Geometry& g, const Tiling& t, const void* phi_in,
                                          void* phi_out, const void* pi_in, void* pi_out, const StepCoef64* k,
                                          bool diag, WavePartial* partials, const DiagCoef& dc, int halo,
                                          hipStream_t s);

template <typename R>
hipError_t launch_blk2d_p(int steps, const BlkShape& b, const Geometry& g, const void* phi_in, void* phi_out,
                          const void* pi_in, void* pi_out, const StepCoef64* k, hipStream_t s)
{
    return launch_blk_r<R>(steps, b, g, phi_in, phi_out, pi_in, pi_out, k, s);
}

template hipError_t launch_blk2d_p<PRS_REAL>(int steps, const BlkShape& b, const Geometry& g, const void* phi_in,
                                             void* phi_out, const void* pi_in, void* pi_out, const StepCoef64* k,
                                             hipStream_t s);

}  // namespace prs
