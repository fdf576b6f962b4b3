// Matrix-core decode kernels over bf16 caches for score widths 33 to 64.
#include "rap_decode_bf16.h"

namespace rap {

hipError_t launch_decode_bf16_k2(const DecodeArgs& a, hipStream_t stream) { return launch_k<2>(a, stream); }

}  // namespace rap
