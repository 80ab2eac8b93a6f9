// Dslash, FP16S with FP32 output: instances of dslash_kernel.h.
#include "dslash_kernel.h"

namespace hisq {

template int launch_epi<H16, H16, F32>(const Geom &g, const DslashLaunch &a, hipStream_t s);

}  // namespace hisq
