// Tile quantizer for head_dim 128, and the choice between it and the other head dimensions.
// The kernels are in quantize_tile.h.
#include "quantize_tile.h"

namespace cq {

bool quantize_tuned_supported(int rows, int n_vis, int d, int bits, int axis, int group) {
  if ((d != 64 && d != 128 && d != 256) || n_vis <= 0 || group < 1) return false;
  if (bits != 1 && bits != 2 && bits != 4 && bits != 8) return false;
  if (axis == CQ_AXIS_CHANNEL ? n_vis % group != 0
                              : axis != CQ_AXIS_TOKEN || group > d || (group != 32 && group != 64 && group != 128 && group != 256))
    return false;
  return launchable(make_task(nullptr, cq_qtensor_t{}, (size_t)rows * (size_t)n_vis, bits, axis, group));
}

hipError_t launch_quantize_tuned(const QuantizeJob* jobs, int n_jobs, int rows, int n_vis, int d, int bits,
                                 hipStream_t stream) {
  const size_t n_tokens = (size_t)rows * (size_t)n_vis;
  if (d == 128) return launch_quantize_dim<128>(jobs, n_jobs, n_tokens, bits, stream);
  if (d == 64) return launch_quantize_64(jobs, n_jobs, n_tokens, bits, stream);
  if (d == 256) return launch_quantize_256(jobs, n_jobs, n_tokens, bits, stream);
  return hipErrorInvalidValue;
}

}  // namespace cq
