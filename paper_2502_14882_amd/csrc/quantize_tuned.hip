// Tile quantizer for head_dim 128, and the choice between it and the other head dimensions.
// The kernels are in quantize_tile.h.
#include "quantize_tile.h"

namespace cq {

bool quantize_tuned_supported(int n_vis, int d, int bits, int axis, int group) {
  if ((d != 64 && d != 128 && d != 256) || n_vis <= 0 || group < 1) return false;
  if (bits != 1 && bits != 2 && bits != 4 && bits != 8) return false;
  if (axis == CQ_AXIS_CHANNEL) return n_vis % group == 0;
  if (axis != CQ_AXIS_TOKEN) return false;
  return group <= d && (group == 32 || group == 64 || group == 128 || group == 256);
}

hipError_t launch_quantize_tuned(const void* x_f16, const cq_qtensor_t& out, int rows, int n_vis,
                                 int d, int bits, int axis, int group, hipStream_t stream) {
  const size_t n_tokens = (size_t)rows * (size_t)n_vis;
  if (d == 128) return launch_quantize_dim<128>(x_f16, out, n_tokens, bits, axis, group, stream);
  return launch_quantize_heads(x_f16, out, n_tokens, d, bits, axis, group, stream);
}

}  // namespace cq
