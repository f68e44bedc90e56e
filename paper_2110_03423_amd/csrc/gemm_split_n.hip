// Split products, op(A) = A.
#include "gemm_split.hpp"

namespace rsvd {
hipError_t split_by_tile_n(hipStream_t s, const GemmParams &P, int batch, char *packed) {
  return split_by_tile<false>(s, P, batch, packed);
}
hipError_t split_init_n() { return split_init<false>(); }
}  // namespace rsvd
