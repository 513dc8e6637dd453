// prs_adjoint3d.hip -- the adjoint's 3D LDS reverse passes, for the field
// precision PRS_REAL (float or double) this translation unit is compiled for;
// the device templates are in prs_device.h.

#include "prs_device.h"

#ifndef PRS_REAL
#error "compile with -DPRS_REAL=float or -DPRS_REAL=double"
#endif

namespace prs {

template <typename R>
hipError_t launch_tba3l_p(int T, const Geometry& g, const Tiling& t, const void* w_in, void* w_out,
                          const void* mu_in, void* mu_out, const void* const* phi, double* gacc, const AdjCoef64* c,
                          hipStream_t s)
{
    return launch_tba3l_r<R>(T, g, t, w_in, w_out, mu_in, mu_out, phi, gacc, c, s);
}

template hipError_t launch_tba3l_p<PRS_REAL>(int T, const Geometry& g, const Tiling& t, const void* w_in, void* w_out,
                                             const void* mu_in, void* mu_out, const void* const* phi, double* gacc,
                                             const AdjCoef64* c, hipStream_t s);

}  // namespace prs
