// Dispatch of the shared-link multi-RHS Dslash (kernel: dslash_shared.h; one
// source file per set of formats holds its instances).

#include "solver_internal.h"

namespace hisq {

template <int LF, int SI, int SO>
int launch_shared_fmt(const Geom &g, const DslashLaunch &a, hipStream_t s);
extern template int launch_shared_fmt<F64, F64, F64>(const Geom &g, const DslashLaunch &a, hipStream_t s);
extern template int launch_shared_fmt<F32, F32, F32>(const Geom &g, const DslashLaunch &a, hipStream_t s);
extern template int launch_shared_fmt<H16, H16, H16>(const Geom &g, const DslashLaunch &a, hipStream_t s);
extern template int launch_shared_fmt<H16, H16, F32>(const Geom &g, const DslashLaunch &a, hipStream_t s);
extern template int launch_shared_fmt<H16, F32, F32>(const Geom &g, const DslashLaunch &a, hipStream_t s);

int launch_dslash_shared(const Geom &g, const DslashLaunch &a, hipStream_t s) {
    if (!order_supported(g, a.order, a.block) || !a.tiles) {
        set_error("dslash: shared launch shape not supported for this lattice");
        return HISQ_ERR_INVALID;
    }
    int rc = -1;
    if (a.fmt_links == F64 && a.fmt_in == F64 && a.fmt_out == F64) rc = launch_shared_fmt<F64, F64, F64>(g, a, s);
    else if (a.fmt_links == F32 && a.fmt_in == F32 && a.fmt_out == F32) rc = launch_shared_fmt<F32, F32, F32>(g, a, s);
    else if (a.fmt_links == H16 && a.fmt_in == H16 && a.fmt_out == H16) rc = launch_shared_fmt<H16, H16, H16>(g, a, s);
    else if (a.fmt_links == H16 && a.fmt_in == H16 && a.fmt_out == F32) rc = launch_shared_fmt<H16, H16, F32>(g, a, s);
    else if (a.fmt_links == H16 && a.fmt_in == F32 && a.fmt_out == F32) rc = launch_shared_fmt<H16, F32, F32>(g, a, s);
    if (rc != 0) {
        set_error("dslash: unsupported precision / tile combination");
        return HISQ_ERR_UNSUPPORTED;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error(std::string("dslash launch: ") + hipGetErrorString(e));
        return HISQ_ERR_HIP;
    }
    return HISQ_OK;
}

}  // namespace hisq
