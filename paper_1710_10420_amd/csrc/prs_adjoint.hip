// prs_adjoint.hip -- the adjoint's kernels (recomputation and reverse sweep), for the field precision
// PRS_REAL (float or double) this translation unit is compiled for; the
// device templates are in prs_device.h.  One unit per dimension, direction
// and precision, so that they compile in parallel.

#include "prs_device.h"

#ifndef PRS_REAL
#error "compile with -DPRS_REAL=float or -DPRS_REAL=double"
#endif

namespace prs {

template <typename R>
hipError_t launch_adjoint_p(const Geometry& g, const Tiling& t, const void* w_in, void* w_out, void* mu,
                            const void* phi_n, double* gacc, const AdjCoef64& c, hipStream_t s)
{
    return launch_adjoint_r<R>(g, t, w_in, w_out, mu, phi_n, gacc, c, s);
}

template hipError_t launch_adjoint_p<PRS_REAL>(const Geometry& g, const Tiling& t, const void* w_in, void* w_out,
                                               void* mu, const void* phi_n, double* gacc, const AdjCoef64& c,
                                               hipStream_t s);

template <typename R>
hipError_t launch_tb_all_p(int T, const Geometry& g, const Tiling& t, const void* phi_in, void* const* phi_lv,
                           const void* pi_in, void* pi_out, const StepCoef64* k, hipStream_t s)
{
    return launch_tb_all_r<R>(T, g, t, phi_in, phi_lv, pi_in, pi_out, k, s);
}

template hipError_t launch_tb_all_p<PRS_REAL>(int T, const Geometry& g, const Tiling& t, const void* phi_in,
                                              void* const* phi_lv, const void* pi_in, void* pi_out,
                                              const StepCoef64* k, hipStream_t s);

template <typename R>
hipError_t launch_tba_p(int T, const Geometry& g, const Tiling& t, const void* w_in, void* w_out, const void* mu_in,
                        void* mu_out, const void* const* phi, double* gacc, const AdjCoef64* c, hipStream_t s)
{
    return launch_tba_r<R>(T, g, t, w_in, w_out, mu_in, mu_out, phi, gacc, c, s);
}

template hipError_t launch_tba_p<PRS_REAL>(int T, const Geometry& g, const Tiling& t, const void* w_in, void* w_out,
                                           const void* mu_in, void* mu_out, const void* const* phi, double* gacc,
                                           const AdjCoef64* c, hipStream_t s);

template <typename R>
hipError_t launch_tb_mid_p(int T, const Geometry& g, const Tiling& t, const void* phi_in, void* phi_out,
                           const void* pi_in, void* pi_out, void* phi_mid, void* pi_mid, const StepCoef64* k,
                           hipStream_t s)
{
    return launch_tb_mid_r<R>(T, g, t, phi_in, phi_out, pi_in, pi_out, phi_mid, pi_mid, k, s);
}

template hipError_t launch_tb_mid_p<PRS_REAL>(int T, const Geometry& g, const Tiling& t, const void* phi_in,
                                              void* phi_out, const void* pi_in, void* pi_out, void* phi_mid,
                                              void* pi_mid, const StepCoef64* k, hipStream_t s);

template <typename R>
hipError_t launch_tbf_p(int T, const Geometry& g, const Tiling& t, const void* phi_s, const void* pi_s,
                        const void* w_in, void* w_out, const void* mu_in, void* mu_out, double* gacc,
                        const StepCoef64* k, const AdjCoef64* c, hipStream_t s)
{
    return launch_tbf_r<R>(T, g, t, phi_s, pi_s, w_in, w_out, mu_in, mu_out, gacc, k, c, s);
}

template hipError_t launch_tbf_p<PRS_REAL>(int T, const Geometry& g, const Tiling& t, const void* phi_s,
                                           const void* pi_s, const void* w_in, void* w_out, const void* mu_in,
                                           void* mu_out, double* gacc, const StepCoef64* k, const AdjCoef64* c,
                                           hipStream_t s);

}  // namespace prs
