// Shared-link multi-RHS Dslash, FP64: instances of dslash_shared.h.
#include "dslash_shared.h"

namespace hisq {

template int launch_shared_fmt<F64, F64, F64>(const Geom &g, const DslashLaunch &a, hipStream_t s);

}  // namespace hisq
