// Shared-link multi-RHS Dslash, FP32: instances of dslash_shared.h.
#include "dslash_shared.h"

namespace hisq {

template int launch_shared_fmt<F32, F32, F32>(const Geom &g, const DslashLaunch &a, hipStream_t s);

}  // namespace hisq
