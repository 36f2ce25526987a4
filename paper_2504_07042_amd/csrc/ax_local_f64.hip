// AxLocal kernels in double arithmetic: trilinear elements, full and partial recomputation (the
// other geometry forms are in ax_local_f64_geo.hip, so that the two compile in parallel).
#include "ax_local_impl.h"

namespace ax {

int axl_dispatch_f64_geo(int geo_kind, int N, int64_t E, int nrhs, const double* geo, const double* Gs,
                         const double* X, double* Y, const double* D, const double* xi, const double* w,
                         hipStream_t st, const int32_t* l2g, int64_t ldg, int64_t es, int64_t ccs, FusedOut* fo);

int axl_dispatch_f64(int geo_kind, int N, int64_t E, int nrhs, const double* geo, const double* Gs,
                      const double* X, double* Y, const double* D, const double* xi, const double* w,
                      hipStream_t st, const int32_t* l2g, int64_t ldg, int64_t es, int64_t ccs, FusedOut* fo)
{
    switch (geo_kind) {
    case GEO_TRI: return dispatch<GEO_TRI, double>(N, E, nrhs, geo, Gs, X, Y, D, xi, w, st, l2g, ldg, es, ccs, fo);
    case GEO_TRIL: return dispatch<GEO_TRIL, double>(N, E, nrhs, geo, Gs, X, Y, D, xi, w, st, l2g, ldg, es, ccs, fo);
    default:
        return axl_dispatch_f64_geo(geo_kind, N, E, nrhs, geo, Gs, X, Y, D, xi, w, st, l2g, ldg, es, ccs, fo);
    }
}

}  // namespace ax
