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

// Whether the tile kernels also finish sooner than the shape-agnostic ones.  They do, but for short groups of
// tokens: a group under 128 tokens other than 32 and 64 is a block of 256 threads of its own, which
// derives the parameters and thresholds of every channel for a few tokens, while the other kernel spends
// one thread per channel on it.  Microseconds, one tensor of 128 rows x 4096 tokens, shape-agnostic / tile:
//   128 channels, 1 bit:   4 tokens 161 / 287, 12: 119 / 99, 16: 114 / 77, 31: 114 / 44
//                 2 bits:  4 tokens 144 / 481, 16: 109 / 124, 20: 111 / 100, 24: 112 / 84, 31: 114 / 69
//                 4 bits:  24 tokens 112 / 128, 28: 113 / 111, 31: 116 / 102
//                 8 bits:  1 token 302 / 2605, 16: 115 / 193, 24: 117 / 135, 28: 118 / 118, 31: 122 / 108
//   256 channels, 2 bits:  16 tokens 286 / 260; 8 rows: 13.6 / 19.7, 24: 16.1 / 15.2, 31: 17.5 / 13.1
// The line is where the slower of 8, 64 and 256 rows broke even when 1 and 2 bits took a fifth to a quarter longer on the tile
// kernels (1 bit 12 tokens 118 / 121, 2 bits 20: 111 / 127); since then groups of 12 to 15 tokens of 1 bit and of 20 to 23 of 2 bits stay
// with the slower kernel (8 rows x 14 tokens, 1 bit 10.7 / 8.0, x 20, 2 bits 11.6 / 9.2).
bool quantize_tile_is_faster(int d, int bits, int axis, int group) {
  if (axis == CQ_AXIS_TOKEN) return true;
  const int line = bits == 1 ? 16 : bits == 2 ? 24 : 28;
  return group >= line * (d == 256 ? 9 : 8) / 8;
}

static hipError_t launch_quantize_tiles(const QuantizeJob* jobs, int n_jobs, size_t n_tokens, int d, int bits,
                                        hipStream_t stream) {
  if (d == 128) return launch_quantize_dim<128>(jobs, n_jobs, n_tokens, bits, stream);
  if (d == 64) return launch_quantize_64(jobs, n_jobs, n_tokens, bits, stream);
  if (d == 256) return launch_quantize_256(jobs, n_jobs, n_tokens, bits, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_quantize_tuned(const QuantizeJob* jobs, int n_jobs, int rows, int n_vis, int d, int bits,
                                 hipStream_t stream) {
  const size_t n_tokens = (size_t)rows * (size_t)n_vis;
  // groups that registers hold: both tensors together, or one of them
  bool slices[2] = {false, false};
  for (int i = 0; i < n_jobs; ++i) slices[i] = quantize_slice_supported(n_tokens, d, bits, jobs[i].axis, jobs[i].group);
  if (n_jobs == 2 && slices[0] && slices[1] && jobs[0].group == jobs[1].group)
    return launch_quantize_slices(jobs, 2, n_tokens, d, bits, stream);
  if (slices[0] || slices[1]) {
    for (int i = 0; i < n_jobs; ++i) {
      const hipError_t e = slices[i] ? launch_quantize_slices(&jobs[i], 1, n_tokens, d, bits, stream)
                                     : launch_quantize_tiles(&jobs[i], 1, n_tokens, d, bits, stream);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  return launch_quantize_tiles(jobs, n_jobs, n_tokens, d, bits, stream);
}

}  // namespace cq
