// Prefill attention kernels for score widths d_k in (32, 64] (KS = 2 fragments of 32).
#include "rap_prefill_kernel.h"

namespace rap {

hipError_t launch_prefill_ks2(const PrefillArgs& a, hipStream_t stream) { return launch_prefill_k<2>(a, stream); }

}  // namespace rap
