// Products of fp64 operands: narrow ones with A^T by gemm_stream.hpp, gemm_pipe.hpp where their rows are 16-byte pieces and there is
// no centring, else gemm_impl.hpp.
#include "gemm_pipe.hpp"
#include "gemm_stream.hpp"

namespace rsvd {
size_t gemm_partial_bytes_f64(const rsvd_ctx *ctx, int64_t M, int64_t N, int64_t K, int trans_a) {
  return GemmDispatch<double, double, double>::partial_bytes(ctx, M, N, K, trans_a != 0);
}

// (chains: tiles of products with up to 128 columns)
#define RSVD_PIPE_TILES(X) X(64, 16, 4, 1, true) X(64, 32, 4, 1, true) X(64, 48, 4, 1, true) X(64, 64, 4, 1, true) X(64, 80, 4, 1, true) \
  X(64, 96, 4, 1, true) X(64, 112, 4, 1, true) X(64, 128, 4, 1, true) X(64, 64, 4, 1, false) X(64, 80, 4, 1, false) X(64, 96, 4, 1, false) \
  X(128, 64, 2, 2, false) X(128, 96, 2, 2, false)

template <bool TA>
static hipError_t pipe_by_tile(hipStream_t s, const GemmParams &P, int bm, int bn, bool chains, int batch) {
#define RSVD_PIPE(BM, BN, WGM, WGN, CHAINS) \
  if (bm == BM && bn == BN && chains == CHAINS) return PipeRun<TA, BM, BN, WGM, WGN, CHAINS>::go(s, P, batch);
  RSVD_PIPE_TILES(RSVD_PIPE)
#undef RSVD_PIPE
  return hipErrorInvalidValue;
}

// Below 10^7 multiply-adds (the blocks of a Cholesky factorisation) either kernel waits for its first loads.
hipError_t gemm_launch_f64(rsvd_ctx *ctx, hipStream_t s, const GemmDesc &d) {
  if (d.M <= 0 || d.N <= 0) return hipSuccess;
  if (stream_takes<double>(d)) return stream_launch<double>(ctx, s, d);
  const double madds = (double)d.M * (double)d.N * (double)d.K * (double)d.batch;
  if (madds < 1e7 || !pipe_can(d)) return GemmDispatch<double, double, double>::launch(ctx, s, d);
  return pipe_launch(ctx, s, d, [&](const GemmParams &P, int bm, int bn, bool chains) {
    return d.trans_a ? pipe_by_tile<true>(s, P, bm, bn, chains, d.batch) : pipe_by_tile<false>(s, P, bm, bn, chains, d.batch);
  });
}
}  // namespace rsvd
