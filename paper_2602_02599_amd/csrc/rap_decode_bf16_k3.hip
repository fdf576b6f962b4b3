// Matrix-core decode kernels over bf16 caches for score widths 65 to 96.
#include "rap_decode_bf16.h"

namespace rap {

hipError_t launch_decode_bf16_k3(const DecodeArgs& a, hipStream_t stream) { return launch_k<3>(a, stream); }

}  // namespace rap
