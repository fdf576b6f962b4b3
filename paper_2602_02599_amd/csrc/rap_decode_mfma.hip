// Dispatch of the matrix-core decode kernel (rap_decode_kernel.h) on the kind of cache and the score width,
// and the LDS size it needs.
#include "rap_decode_kernel.h"

namespace rap {

hipError_t launch_decode_bf16_k1(const DecodeArgs& a, hipStream_t stream);   // rap_decode_bf16_k1.hip .. _k4.hip
hipError_t launch_decode_bf16_k2(const DecodeArgs& a, hipStream_t stream);
hipError_t launch_decode_bf16_k3(const DecodeArgs& a, hipStream_t stream);
hipError_t launch_decode_bf16_k4(const DecodeArgs& a, hipStream_t stream);
hipError_t launch_decode_mfma_q8(const DecodeArgs& a, hipStream_t stream);   // rap_decode_mfma_q8.hip
hipError_t launch_decode_mfma_mx4(const DecodeArgs& a, hipStream_t stream);  // rap_decode_mfma_mx4.hip

// LDS bytes one wavefront needs: its K tile, its V tile and slack for the fragment reads that run
// past the last row, or the hand-over area of the final fold, whichever is larger.
// (4-bit caches: the V tile's scale bytes and codes; a lane beyond the row's channels reads past it.)
int mfma_lds_wave_bytes(int d_k, int d_v, bool q8, int cols, bool mx4) {
  const int nt = mx4 ? mx4_lane_channels(mx_blocks(d_v)) : decode_v_tiles(d_v, q8);
  const int tiles = mx4 ? 32 * (4 + 16 * mx_blocks(d_v)) + 128
                        : 1024 * (k_tile_loads((d_k + 31) / 32, q8) + v_tile_loads(nt, q8)) + 128;
  const int fold = (32 + (cols > kMaxGroup ? kMaxCols : kMaxGroup) * 16 * nt) * 4;
  const int need = tiles > fold ? tiles : fold;
  return (need + 127) / 128 * 128;
}

hipError_t launch_decode_mfma(const DecodeArgs& a, hipStream_t stream) {
  if (a.k_scales4 != nullptr) return launch_decode_mfma_mx4(a, stream);
  if (a.k_scale != nullptr) return launch_decode_mfma_q8(a, stream);
  switch ((a.d_k + 31) / 32) {
    case 1: return launch_decode_bf16_k1(a, stream);
    case 2: return launch_decode_bf16_k2(a, stream);
    case 3: return launch_decode_bf16_k3(a, stream);
    case 4: return launch_decode_bf16_k4(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace rap
