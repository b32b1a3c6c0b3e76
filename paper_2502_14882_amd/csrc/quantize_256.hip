// Tile quantizer for head_dim 256 (a file of its own: it compiles beside the others).  The kernels are
// in quantize_tile.h.
#include "quantize_tile.h"

namespace cq {

hipError_t launch_quantize_256(const QuantizeJob* jobs, int n_jobs, size_t n_tokens, int bits,
                               hipStream_t stream) {
  return launch_quantize_dim<256>(jobs, n_jobs, n_tokens, bits, stream);
}

}  // namespace cq
