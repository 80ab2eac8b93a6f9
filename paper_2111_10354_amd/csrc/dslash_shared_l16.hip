// Shared-link multi-RHS Dslash, FP16 links on FP32 vectors: instances of dslash_shared.h.
#include "dslash_shared.h"

namespace hisq {

template int launch_shared_fmt<H16, F32, F32>(const Geom &g, const DslashLaunch &a, hipStream_t s);

}  // namespace hisq
