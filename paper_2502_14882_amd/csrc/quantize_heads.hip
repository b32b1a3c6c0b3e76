// Tile quantizer for head_dim 64 and 256 (a file of its own: the two compile beside the
// head_dim 128 kernels).  The kernels are in quantize_tile.h.
#include "quantize_tile.h"

namespace cq {

hipError_t launch_quantize_heads(const void* x_f16, const cq_qtensor_t& out, size_t n_tokens, int d,
                                 int bits, int axis, int group, hipStream_t stream) {
  if (d == 64) return launch_quantize_dim<64>(x_f16, out, n_tokens, bits, axis, group, stream);
  if (d == 256) return launch_quantize_dim<256>(x_f16, out, n_tokens, bits, axis, group, stream);
  return hipErrorInvalidValue;
}

}  // namespace cq
