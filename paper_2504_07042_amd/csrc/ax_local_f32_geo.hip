// AxLocal kernels in float arithmetic: parallelepipeds, stored factors and the Helmholtz form.
#include "ax_local_impl.h"

namespace ax {

int axl_dispatch_f32_geo(int geo_kind, int N, int64_t E, int nrhs, const double* geo, const float* Gs,
                         const float* X, float* Y, const double* D, const double* xi, const double* w,
                         hipStream_t st, const int32_t* l2g, int64_t ldg, int64_t es, int64_t ccs, FusedOut* fo)
{
    switch (geo_kind) {
    case GEO_PARA: return dispatch<GEO_PARA, float>(N, E, nrhs, geo, Gs, X, Y, D, xi, w, st, l2g, ldg, es, ccs, fo);
    case GEO_HELM: return dispatch<GEO_HELM, float>(N, E, nrhs, geo, Gs, X, Y, D, xi, w, st, l2g, ldg, es, ccs, fo);
    default: return dispatch<GEO_STORED, float>(N, E, nrhs, geo, Gs, X, Y, D, xi, w, st, l2g, ldg, es, ccs, fo);
    }
}

}  // namespace ax
