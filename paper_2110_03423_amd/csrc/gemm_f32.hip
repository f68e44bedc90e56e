// Products of fp32 operands: on the bf16 matrix cores with split operands (gemm_split.hpp) where there is enough work for
// that, else on the fp32 matrix cores (gemm_impl.hpp).
#include "gemm_split.hpp"

namespace rsvd {
size_t gemm_partial_bytes_f32(const rsvd_ctx *ctx, int64_t M, int64_t N, int64_t K, int trans_a) {
  return GemmDispatch<float, float, float>::partial_bytes(ctx, M, N, K, trans_a != 0);
}

hipError_t gemm_split_init_device(rsvd_ctx *ctx) {
  (void)ctx;
  const hipError_t e = split_init_n();
  return e == hipSuccess ? split_init_t() : e;
}

// Which products are split.  Up to 32 columns both kernels wait for memory and the fp32 one needs no conversion (65536 x
// 16384, l = 16: 5.7 TB/s).  Below 2^29 multiply-adds (2000 x 500, l = 33: 19 us split, 14 us not) the longer prologue of the
// large tiles costs more than the faster instruction brings; above, split products win from 10000 x 2000, l = 80 (48 -> 41 us)
// to 65536 x 16384, l = 576 (9.2 -> 5.8 ms).
// A triangular B (the applies of R^-1) leaves only part of a short k range per column tile, and the fp32 kernel's narrower tiles
// waste less of it (65536 x 576: 176 us, split 224 us) unless it is down to scalar loads (50021 x 210: 86 us, split 72 us).
static bool takes_split(const GemmDesc &d) {
  const bool aligned = ((uintptr_t)d.A | (uintptr_t)d.B) % 16 == 0 && (d.lda | d.ldb | d.K | d.N) % 4 == 0;
  if (d.b_upper != 0 && aligned) return false;
  return d.N > 32 && (double)d.M * (double)d.N * (double)d.K * (double)d.batch >= 536870912.0 && !d.upper_only &&
         d.alpha == 1.0 && d.beta == 0.0 && split_fits(d.lda, d.ldb);
}

// The packed operand pays from two column tiles on; with one, whichever kernel reads the fp32 operand reads it about as often
// as the packed one would be read, and the extra launch stays (20000 x 5000, l = 128: 205 us either way).
size_t gemm_packed_bytes(int64_t K, int64_t N) { return N > 128 ? split_packed_bytes(K, N) : 0; }

// The number of k ranges that leaves the shortest longest queue of k-tiles on a CU, at most `most`; a range costs about
// four k-tiles more for its prologue and its share of the partial sums.
static SplitChoice split_ranges(const rsvd_ctx *ctx, const GemmDesc &d, int bn, int most) {
  const int64_t tiles = ceil_div(d.M, split_tile_m(bn)) * ceil_div(d.N, bn) * d.batch, ktiles = ceil_div(d.K, kSplitBK);
  const int64_t places = (int64_t)ctx->cu_count * split_wgs_per_cu(bn);
  int64_t best = 1, best_cost = -1;
  for (int64_t s = 1; s <= most && s <= ktiles; ++s) {
    const int64_t per = ceil_div(ktiles, s), ranges = ceil_div(ktiles, per);
    const int64_t cost = ceil_div(tiles * ranges, places) * (per + 4) + (s > 1 ? 2 : 0);
    if (best_cost < 0 || cost < best_cost) { best = s; best_cost = cost; }
  }
  SplitChoice c;
  c.k_per_split = ceil_div(ktiles, best) * kSplitBK;
  c.splits = (int)ceil_div(d.K, c.k_per_split);
  return c;
}

hipError_t gemm_launch_f32(rsvd_ctx *ctx, hipStream_t s, const GemmDesc &d) {
  if (d.M <= 0 || d.N <= 0) return hipSuccess;
  if (!takes_split(d)) return GemmDispatch<float, float, float>::launch(ctx, s, d);
  if (d.batch < 1 || d.batch > 65535) return hipErrorInvalidValue;
  if (d.a_shift != nullptr && (d.dead != nullptr || d.trans_c || d.batch != 1)) return hipErrorInvalidValue;
  const size_t pack = gemm_packed_bytes(d.K, d.N);
  char *packed = (char *)(pack > 0 && d.batch == 1 && d.packed_bytes >= pack ? d.packed : nullptr);
  // the k ranges of the fp32 kernel bound those taken here: the workspace is sized for their partial sums
  const TileChoice t = choose_tile(d.M, d.N, d.K, sizeof(float), d.trans_a != 0);
  SplitChoice c = choose_split(ctx, t, d.M, d.N, d.K, d.force_splits, false, d.batch);
  if (d.force_splits <= 0) c = split_ranges(ctx, d, split_tile_n(d.N), c.splits);
  if (c.splits > 1) {
    const size_t need = (size_t)c.splits * (size_t)d.M * (size_t)d.N * sizeof(float);
    if (d.partial == nullptr || d.partial_bytes < need) return hipErrorInvalidValue;
  }
  const GemmParams P = make_params(d, c);
  hipError_t e;
  {
    ProfScope ps(ctx, s, d.prof_kind);
    e = d.trans_a ? split_by_tile_t(s, P, d.batch, packed) : split_by_tile_n(s, P, d.batch, packed);
  }
  if (e != hipSuccess) return e;
  return finish_splits<float, float, float>(ctx, s, d, P);
}
}  // namespace rsvd
