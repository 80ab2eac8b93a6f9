// Shared-link multi-RHS Dslash, FP16S: instances of dslash_shared.h.
#include "dslash_shared.h"

namespace hisq {

template int launch_shared_fmt<H16, H16, H16>(const Geom &g, const DslashLaunch &a, hipStream_t s);

}  // namespace hisq
