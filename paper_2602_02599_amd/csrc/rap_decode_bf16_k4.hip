// Matrix-core decode kernels over bf16 caches for score widths 97 to 128.
#include "rap_decode_bf16.h"

namespace rap {

hipError_t launch_decode_bf16_k4(const DecodeArgs& a, hipStream_t stream) { return launch_k<4>(a, stream); }

}  // namespace rap
