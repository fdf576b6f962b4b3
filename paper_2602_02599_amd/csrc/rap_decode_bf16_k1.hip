// Matrix-core decode kernels over bf16 caches for score widths up to 32.
#include "rap_decode_bf16.h"

namespace rap {

hipError_t launch_decode_bf16_k1(const DecodeArgs& a, hipStream_t stream) { return launch_k<1>(a, stream); }

}  // namespace rap
