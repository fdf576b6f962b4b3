// Prefill attention kernels for score widths d_k in (96, 128] (KS = 4 fragments of 32).
#include "rap_prefill_kernel.h"

namespace rap {

hipError_t launch_prefill_ks4(const PrefillArgs& a, hipStream_t stream) { return launch_prefill_k<4>(a, stream); }

}  // namespace rap
