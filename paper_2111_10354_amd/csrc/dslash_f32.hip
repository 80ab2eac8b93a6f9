// Dslash, FP32: instances of dslash_kernel.h.
#include "dslash_kernel.h"

namespace hisq {

template int launch_epi<F32, F32, F32>(const Geom &g, const DslashLaunch &a, hipStream_t s);

}  // namespace hisq
