// Split products, op(A) = A^T.
#include "gemm_split.hpp"

namespace rsvd {
hipError_t split_by_tile_t(hipStream_t s, const GemmParams &P, int batch, char *packed) {
  return split_by_tile<true>(s, P, batch, packed);
}
hipError_t split_init_t() { return split_init<true>(); }
}  // namespace rsvd
