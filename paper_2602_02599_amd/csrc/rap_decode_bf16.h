// Dispatch of the matrix-core decode kernel over bf16 caches on the V width, included by one source file
// per score width (rap_decode_bf16_k1.hip .. _k4.hip) so that they compile side by side.
#ifndef RAP_DECODE_BF16_H_
#define RAP_DECODE_BF16_H_

#include "rap_decode_kernel.h"

namespace rap {

namespace {

template <int KCH, int NT, bool VPAIR>
hipError_t launch_inst(const DecodeArgs& a, hipStream_t stream) {
  if (a.block_table != nullptr) return launch_inst2<KCH, NT, VPAIR, true, false>(a, stream);
  return launch_inst2<KCH, NT, VPAIR, false, false>(a, stream);
}

template <int KCH>
hipError_t launch_k(const DecodeArgs& a, hipStream_t stream) {
  const int nt = decode_v_tiles(a.d_v, false);
  if ((a.d_v & 1) == 0 && (nt & 1) == 0) {   // paired 4-byte V reads
    switch (nt) {
      case 2: return launch_inst<KCH, 2, true>(a, stream);
      case 4: return launch_inst<KCH, 4, true>(a, stream);
      case 6: return launch_inst<KCH, 6, true>(a, stream);
      case 8: return launch_inst<KCH, 8, true>(a, stream);
      default: return hipErrorInvalidValue;
    }
  }
  switch (nt) {
    case 1: return launch_inst<KCH, 1, false>(a, stream);
    case 2: return launch_inst<KCH, 2, false>(a, stream);
    case 3: return launch_inst<KCH, 3, false>(a, stream);
    case 4: return launch_inst<KCH, 4, false>(a, stream);
    case 5: return launch_inst<KCH, 5, false>(a, stream);
    case 6: return launch_inst<KCH, 6, false>(a, stream);
    case 7: return launch_inst<KCH, 7, false>(a, stream);
    case 8: return launch_inst<KCH, 8, false>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

}  // namespace rap

#endif  // RAP_DECODE_BF16_H_
