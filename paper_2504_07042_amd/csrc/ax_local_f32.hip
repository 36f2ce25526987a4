// AxLocal kernels in float arithmetic: trilinear elements, full and partial recomputation (the
// other geometry forms are in ax_local_f32_geo.hip, so that the two compile in parallel).
#include "ax_local_impl.h"

namespace ax {

int axl_dispatch_f32_geo(int geo_kind, int N, int64_t E, int nrhs, const double* geo, const float* Gs,
                         const float* X, float* Y, const double* D, const double* xi, const double* w,
                         hipStream_t st, const int32_t* l2g, int64_t ldg, int64_t es, int64_t ccs, FusedOut* fo);

int axl_dispatch_f32(int geo_kind, int N, int64_t E, int nrhs, const double* geo, const float* Gs,
                      const float* X, float* Y, const double* D, const double* xi, const double* w,
                      hipStream_t st, const int32_t* l2g, int64_t ldg, int64_t es, int64_t ccs, FusedOut* fo)
{
    switch (geo_kind) {
    case GEO_TRI: return dispatch<GEO_TRI, float>(N, E, nrhs, geo, Gs, X, Y, D, xi, w, st, l2g, ldg, es, ccs, fo);
    case GEO_TRIL: return dispatch<GEO_TRIL, float>(N, E, nrhs, geo, Gs, X, Y, D, xi, w, st, l2g, ldg, es, ccs, fo);
    default:
        return axl_dispatch_f32_geo(geo_kind, N, E, nrhs, geo, Gs, X, Y, D, xi, w, st, l2g, ldg, es, ccs, fo);
    }
}

}  // namespace ax
