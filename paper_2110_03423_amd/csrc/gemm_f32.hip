// Products of fp32 operands: on the bf16 matrix cores with split operands (gemm_split.hpp) where there is enough work for
// that, narrow ones with A^T by gemm_stream.hpp, else on the fp32 matrix cores (gemm_impl.hpp).
#include "gemm_split.hpp"
#include "gemm_stream.hpp"

namespace rsvd {
size_t gemm_partial_bytes_f32(const rsvd_ctx *ctx, int64_t M, int64_t N, int64_t K, int trans_a) {
  return GemmDispatch<float, float, float>::partial_bytes(ctx, M, N, K, trans_a != 0);
}

hipError_t gemm_split_init_device(rsvd_ctx *ctx) {
  (void)ctx;
  const hipError_t e = split_init_n();
  return e == hipSuccess ? split_init_t() : e;
}

// Which products are split, by their shape (times in us, fp32 kernel against split one).  Up to 32 columns (of A^T X: what is left of
// them by gemm_stream_kernel) both kernels wait for memory and the fp32 one needs no conversion (65536 x 16384, l = 16: 5.8 TB/s), and below 2^29 multiply-adds (2000 x 500, l = 33:
// 22, 25) the longer prologue of the large tiles costs more than the faster instruction brings.  Where both operands are aligned for
// 16-byte loads the fp32 kernel also wins on
//  - a k range of a few k-tiles, unless one column tile of 96 to 144 shares the traffic of A: 1000000 x 64, l = 64: 131, 217; 69568 x
//    192, l = 192: 73, 84; but 57504 x 176, l = 112: 45, 38;
//  - up to 48 columns of A X, whose tiles of A are half of all LDS traffic, unless the k range is long (69808 x 464: 53, 58;
//    126064 x 592: 93, 92; 62208 x 1200: 90, 81) and there is work (1872 x 9760: 38, 40; 768 x 30640: 43, 42), and of A^T X with fewer
//    than 96 rows in a tile of 128 (48 x 593552: 75, 90; 96 x 139920: 40, 40);
//  - a triangular B (the applies of R^-1), which leaves only part of a short k range per column tile: its narrower tiles waste less
//    of that (65536 x 576: 176, 224).
// Otherwise: 10000 x 2000, l = 80: 56 -> 47; 50021 x 210, triangular, scalar loads: 86 -> 72; 65536 x 16384, l = 576: 9179 -> 5512.
// A narrow operand of the workspace that is not aligned, which the fp32 kernel reads in 16-byte pieces all the same, counts as one that it
// cannot: the split kernel's error against 64 bits is 2.8 to 5 times smaller, and these rules decide where it is given up.
static bool takes_split(const GemmDesc &d, bool aligned) {
  const double madds = (double)d.M * (double)d.N * (double)d.K * (double)d.batch;
  if (d.N <= 32 || madds < 536870912.0 || d.upper_only || d.alpha != 1.0 || d.beta != 0.0 || !split_fits(d.lda, d.ldb)) return false;
  if (!aligned) return true;
  if (d.b_upper != 0) return false;
  if (d.K < 208 && (d.N < 96 || d.N > 144)) return false;
  if (d.N <= 48) return d.trans_a ? d.M >= 96 : (d.K >= 640 && madds >= 1073741824.0);
  return true;
}
// ... and by how the workgroups fill the chip: a split one takes a CU or half of one for 256 or 128 rows, where the fp32 kernel
// has four smaller ones per CU.  What share of the places has to be taken depends on the k-tiles of a range:
//  six and fewer   0.72 (1168 x 5984, l = 80) 34, 40; 0.59 (336 x 15904, l = 80) 33, 38; 0.78 (256 x 25456, l = 96) 39, 39
//  up to fifteen   0.41 (1696 x 1312, l = 304) 44, 47; 0.55 (17808 x 240, l = 176) 43, 40; A^T X (k from the long side) and ranges that
//                  are not cut: 0.50 (18240 x 256, l = 224) 45, 43; 0.53 (34352 x 240, l = 96) 45, 38
//  more            0.50 (768 x 32848, l = 96) 76, 63; 0.53 (576 x 11328, l = 304) 88, 56
//  scalar loads    0.32 (551 x 2534, l = 413) 43, 52; 0.44 (1220 x 1724, l = 476) 58, 48; not cut: 0.26 (16809 x 407, l = 136) 70, 55
//  l <= 48         0.63 (41145 x 1908, l = 44) 108, 116; 0.83 (62208 x 1200) 90, 81
// A last wave that is nearly empty costs more than the faster instruction brings in narrow products: l = 48, 1.2 waves: 78592 x
// 1200 107, 126; 1.4: 91648 x 4000 366, 361; l = 96, 1.05 waves: 68608 x 400 76, 79; 68608 x 1200 180, 176; l = 128: 68160 x 128
// 43, 56; 68608 x 400 97, 92.  (Over 260 random shapes in both directions the rule is within 1 % of the better kernel each time.)
static bool fills_chip(const rsvd_ctx *ctx, const GemmDesc &d, bool aligned, int bn, const SplitChoice &c) {
  const int64_t wgs = ceil_div(d.M, split_tile_m(bn)) * ceil_div(d.N, bn) * d.batch * c.splits;
  const int64_t places = (int64_t)ctx->cu_count * split_wgs_per_cu(bn), ktiles = c.k_per_split / kSplitBK;
  const bool whole = c.splits == 1;
  const int share = !aligned ? (whole ? 25 : 35) : ktiles <= 6 ? 75 : d.N <= 48 ? 70 : ktiles >= 16 ? 40 : d.trans_a || whole ? 50 : 55;
  if (wgs * 100 < places * share) return false;
  if (!aligned || d.N > 128 || wgs <= places) return true;
  const bool full = wgs * 100 >= ceil_div(wgs, places) * places * 65;
  if (d.N <= 48) return full && d.K >= 2048;
  return full || d.K >= (d.N <= 96 ? 512 : 256);
}

// The packed operand pays from two column tiles on; with one, whichever kernel reads the fp32 operand reads it about as often
// as the packed one would be read, and the extra launch stays (20000 x 5000, l = 128: 205 us either way).  And it pays as long as
// enough row tiles read it: with fewer, what the packing reads and writes is more than it saves (160 x 154432, l = 160: 185 us, split
// in place 102; 1500 x 30000, l = 300, six row tiles: 202, 176; 2244 x 67556, l = 411, nine: 716, 754; 20000 x 5000, l = 576:
// 760, 928).
size_t gemm_packed_bytes(int64_t M, int64_t N, int64_t K) {
  return N > 128 && ceil_div(M, split_tile_m(split_tile_n(N))) >= 8 ? split_packed_bytes(K, N) : 0;
}

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
  typedef GemmDispatch<float, float, float> Plain;
  if (d.M <= 0 || d.N <= 0) return hipSuccess;
  if (stream_takes<float>(d)) return stream_launch<float>(ctx, s, d);
  const bool aligned = Plain::aligned_a(d) && Plain::aligned_b(d);
  if (!takes_split(d, aligned)) return Plain::launch(ctx, s, d);
  if (d.batch < 1 || d.batch > 65535) return hipErrorInvalidValue;
  if (d.a_shift != nullptr && (d.dead != nullptr || d.trans_c || d.batch != 1)) return hipErrorInvalidValue;
  // the k ranges of the fp32 kernel bound those taken here: the workspace is sized for their partial sums
  const TileChoice t = choose_tile(d.M, d.N, d.K, sizeof(float), d.trans_a != 0);
  SplitChoice c = choose_split(ctx, t, d.M, d.N, d.K, d.force_splits, false, d.batch);
  const int bn = split_tile_n(d.N);
  if (d.force_splits <= 0) c = split_ranges(ctx, d, bn, c.splits);
  if (!fills_chip(ctx, d, aligned, bn, c)) return Plain::launch(ctx, s, d);
  if (c.splits > 1) {
    const size_t need = (size_t)c.splits * (size_t)d.M * (size_t)d.N * sizeof(float);
    if (d.partial == nullptr || d.partial_bytes < need) return hipErrorInvalidValue;
  }
  const GemmParams P = make_params(d, c);
  const size_t pack = gemm_packed_bytes(d.M, d.N, d.K);
  char *packed = (char *)(pack > 0 && d.batch == 1 && d.packed_bytes >= pack ? d.packed : nullptr);
  hipError_t e;
  {
    ProfScope ps(ctx, s, d.prof_kind);
    e = d.trans_a ? split_by_tile_t(s, P, d.batch, packed) : split_by_tile_n(s, P, d.batch, packed);
  }
  if (e != hipSuccess) return e;
  return finish_splits<float, float, float>(ctx, s, d, P);
}
}  // namespace rsvd
