// Products C = op(A) B of fp64 operands that have 16-byte rows, with k-tiles that go from memory to LDS without touching a register.
//
// gemm_kernel (gemm_impl.hpp) loads a k-tile into registers, writes it to LDS between two barriers and hides what that costs behind four
// or five workgroups per CU.  In fp64 with 48 columns and more it kept the matrix pipe busy for half of the time (a matrix instruction
// takes 64 cycles, but the wavefronts of a workgroup read their operands all at once behind a barrier), and the ~1000 k ranges that such
// a grid wants write and read partial sums of a third of A.  Here a workgroup has a ring of S k-tiles of 128 bytes of k each in LDS,
// filled by loads that write there themselves: one barrier per k-tile, no staging registers, k-tiles half as deep.  Calls of
// rsvd_stage_gemm_an / _atn in us, gemm_kernel -> this:
//   5000 x 5000, l = 64      113 -> 86, 107 -> 85          8000 x 2000, l = 210     211 -> 148, 207 -> 146
//   30000 x 1000, l = 48     103 -> 78, 98 -> 78           12000 x 9000, l = 200    1028 -> 905, 1113 -> 958
//   20000 x 10000, l = 96    790 -> 699, 941 -> 709        20000 x 20000, l = 288   4296 -> 3643, 3964 -> 3755 (63, 61 TFLOP/s)
// Up to 16 columns, where memory is the bound, about the same (3000 x 20000, l = 16: 112 -> 101, 104 -> 107; 1624 x 39874, l = 14: 113 -> 123,
// 111 -> 108).
// What was tried: four more k-tiles in flight with two workgroups per CU (5 to 12 % slower at l = 48 and 64 than four workgroups with one
// k-tile ahead); the work dealt out evenly in k-tiles, sums of shared tiles added behind (the loop that crosses tiles costs more than the
// last wave: 3.83 -> 3.97 ms at l = 288, with 64-row tiles 4.4); fp32 operands, narrow (no gain: l = 32 within 3 %, l = 48 5 to 15 % slower
// than the split products) and summed in fp64 (Gram matrices of 65536 x 576: 8 % slower).
//
// LDS is written in the order of the lanes, 16 bytes each, so a layout is chosen by which piece of memory a lane fetches:
//   [row][k] tiles (A as stored): 128 bytes a row, the eight pieces of row r in places piece ^ (r / 2 mod 8): sixteen lanes that read
//     the same k of sixteen rows, 16 bytes each, meet every bank once;
//   [k][column] tiles (B, and A for A^T): a lane's 16 bytes down a row of A are V consecutive k, one for each of V matrix
//     instructions, so the lanes of instruction (t, e) need the rows k = 4 V t + V kq + e, kq = 0 ... 3: these lie next to each other (row
//     4 V t + 4 e + kq), their pieces exchanged by kq where the row length would bring them to the same banks.
#pragma once

#include "gemm_impl.hpp"

namespace rsvd {

// Workgroups that share a CU, and the k-tiles each has room for (in the 64 KB that a launch may ask for without more ado).  chains: with a
// second set of accumulators, for which the wider tiles take the registers of a workgroup.
constexpr int pipe_wgs(int bm, int bn, bool chains) {
  if (bm > 64 || bn <= 16) return 2;
  return chains ? (bn <= 80 ? 4 : bn <= 112 ? 3 : 2) : bn <= 96 ? 4 : 3;
}
constexpr int pipe_stages(int bm, int bn, bool chains) {
  const int wgs = pipe_wgs(bm, bn, chains), kb = 160 / wgs < 64 ? 160 / wgs : 64;
  return kb * 1024 / ((bm + bn) * 128);
}

constexpr int kPipeV = 2, kPipeBK = 16;      // elements of a piece, depth of a k-tile

// Operand of s_waitcnt: at most n vector memory operations outstanding, no LDS operation.
constexpr int pipe_wait(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0070; }

// Place of piece `ch` in a row of a [k][column] tile of X columns: sixteen lanes read 128 bytes of it, and rows of a multiple of 256 bytes
// begin at the same bank.
template <int X> __device__ __forceinline__ int pipe_place(int ch, int kq) { return X % 32 == 0 ? ch ^ ((kq & 1) << 3) : ch; }

// The loads of one operand tile of a k-tile, ROWS x BK or BK x ROWS elements, by four wavefronts.
//   KMAJOR: consecutive elements of the stored matrix run along the rows / columns of the tile, k from row to row of the matrix.
// The addresses are one for the workgroup and 32-bit offsets of the lanes (pipe_can sees to it that these suffice): with 64-bit addresses
// of their own the accumulators of the 80 to 112 column tiles no longer fit into the registers.
template <int ROWS, bool KMAJOR> struct PipeLoad {
  static constexpr int V = kPipeV, BK = kPipeBK;
  static constexpr int BYTES = ROWS * 128, PIECES = BYTES / 1024, N = (PIECES + 3) / 4;       // of 1024 bytes; per wavefront
  const char *base;          // element (0, 0) of the next tile
  uint32_t off[N];
  // First k of the 16 bytes inside the tile that lie at place q, and their row (column).
  static __device__ __forceinline__ void place(int q, int &k, int &x) {
    if (KMAJOR) {
      constexpr int PER = ROWS / V;
      const int rp = q / PER, kq = rp & 3;
      x = pipe_place<ROWS>(q - rp * PER, kq) * V;
      k = (rp / (4 * V)) * (4 * V) + V * kq + ((rp >> 2) & (V - 1));
    } else {
      x = q >> 3;
      k = ((q & 7) ^ ((x >> 1) & 7)) * V;
    }
  }
  // extent: rows (columns) that exist; those beyond are read as another one, and not stored.
  __device__ __forceinline__ void init(const double *origin, int64_t ld, int extent, int wave, int lane) {
    base = reinterpret_cast<const char *>(origin);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      int k, x;
      place(piece(wave, i) * 64 + lane, k, x);            // place in LDS, 16 bytes each
      off[i] = (uint32_t)sizeof(double) * (KMAJOR ? (uint32_t)k * (uint32_t)ld + (uint32_t)(x < extent ? x : 0)
                                             : (uint32_t)(x < extent ? x : extent - 1) * (uint32_t)ld + (uint32_t)k);
    }
  }
  static __device__ __forceinline__ int piece(int wave, int i) {
    const int p = wave + 4 * i;
    return PIECES % 4 == 0 || p < PIECES ? p : PIECES - 1;       // (left over: the last piece once more)
  }
  __device__ __forceinline__ void load(char *lds, int wave, int i, uint32_t at) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(base + at),
                                     (__attribute__((address_space(3))) void *)(lds + piece(wave, i) * 1024), 16, 0, 0);
  }
  // k_left: k of the tile that exist (others are read as k = 0, and cleared before they are used)
  __device__ __forceinline__ void issue(char *lds, int64_t ld, int k_left, int wave, int lane) {
    if (k_left >= BK) {
#pragma unroll
      for (int i = 0; i < N; ++i) load(lds, wave, i, off[i]);
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        int k, x;
        place(piece(wave, i) * 64 + lane, k, x);
        load(lds, wave, i, k >= k_left ? off[i] - (uint32_t)sizeof(double) * (uint32_t)k * (KMAJOR ? (uint32_t)ld : 1u) : off[i]);
      }
    }
    base += (KMAJOR ? BK * ld : BK) * (int64_t)sizeof(double);
  }
  // The k from k_left on of a tile in LDS become zero.
  static __device__ __forceinline__ void clear(char *lds, int k_left, int tid) {
    for (int q = tid; q < BYTES / 16; q += 256) {
      int k, x;
      place(q, k, x);
      double *at = reinterpret_cast<double *>(lds + q * 16);
#pragma unroll
      for (int e = 0; e < V; ++e)
        if ((KMAJOR ? k : k + e) >= k_left) at[e] = 0.0;
    }
  }
};

template <int BM, int BN, int S> struct PipeCfg {
  static constexpr int STAGE = (BM + BN) * 128;
  static constexpr size_t lds = (size_t)S * STAGE;
};

// CHAINS: sums of k_chain terms, one after the other into one accumulator, are added up in a second set of accumulators.
template <bool TA, int BM, int BN, int WGM, int WGN, int S, int EPI, bool CHAINS>
__global__ __launch_bounds__(256, pipe_wgs(BM, BN, CHAINS)) void gemm_pipe_kernel(const GemmParams P0) {
  const GemmParams P = select_problem(P0);
  if (P.skip_now) return;
  static_assert(WGM * WGN == 4, "four wavefronts per workgroup");
  constexpr int V = kPipeV, BK = kPipeBK, STAGE = PipeCfg<BM, BN, S>::STAGE;
  constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 16, TN = WN / 16;
  typedef double piece_t __attribute__((ext_vector_type(kPipeV)));
  extern __shared__ __attribute__((aligned(16))) char pipe_lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave / WGN) * WM, wn0 = (wave % WGN) * WN;
  const int r16 = lane & 15, kq = lane >> 4;
  int tile_m, tile_n, split;
  tile_of_workgroup(P, tile_m, tile_n, split);
  const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;
  if (P.upper_bm > 0 && n0 + BN <= m0) return;       // symmetric result: this tile mirrors one that is computed
  const int64_t k_begin = (int64_t)split * P.k_per_split;
  int64_t k_end = (k_begin + P.k_per_split < P.K) ? (k_begin + P.k_per_split) : P.K;
  if (P.b_upper != 0 && n0 + BN < k_end) k_end = n0 + BN;      // rows of B from n0 + BN on are zero in these columns
  const int nkt = k_begin < k_end ? (int)((k_end - k_begin + BK - 1) / BK) : 0;
  const int last_k = (int)(k_end - k_begin) - (nkt - 1) * BK;

  f64x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = (f64x4)0.0;
  f64x4 sum[CHAINS ? TM : 1][CHAINS ? TN : 1];
  if constexpr (CHAINS) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) sum[i][j] = (f64x4)0.0;
  }

  PipeLoad<BM, TA> la;
  PipeLoad<BN, true> lb;
  const double *A = (const double *)P.A, *B = (const double *)P.B;
  la.init(TA ? A + k_begin * P.lda + m0 : A + m0 * P.lda + k_begin, P.lda, (int)(P.M - m0 < BM ? P.M - m0 : BM), wave, lane);
  lb.init(B + k_begin * P.ldb + n0, P.ldb, (int)(P.N - n0 < BN ? P.N - n0 : BN), wave, lane);
  constexpr int LOADS = decltype(la)::N + decltype(lb)::N;      // a wavefront's loads per k-tile
  static_assert((S - 2) * LOADS < 64, "the counter of outstanding loads ends at 63");
  int issued = 0;
  auto issue = [&]() {
    // (behind the last tile nothing is loaded: the last iterations wait for everything)
    if (issued < nkt) {
      char *st = pipe_lds + (issued % S) * STAGE;
      const int left = issued + 1 < nkt ? BK : last_k;
      la.issue(st, P.lda, left, wave, lane);
      lb.issue(st + BM * 128, P.ldb, left, wave, lane);
    }
    ++issued;
  };
#pragma unroll
  for (int s = 0; s < S - 1; ++s) issue();

  // offsets of this lane's operands inside a stage
  int a_row[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int row = wm0 + i * 16 + r16;
    a_row[i] = TA ? 0 : row * 128;
  }
  const int a_swz = TA ? 0 : ((wm0 + r16) >> 1) & 7;           // (the same in every block of 16 rows)
  auto column = [&](auto x, int col) {                          // byte offset of column `col` in a [k][column] row read by lanes kq
    constexpr int X = decltype(x)::value;
    return pipe_place<X>(col / V, kq) * 16 + (col % V) * (int)sizeof(double);
  };
  int a_col[TM], b_col[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) a_col[i] = TA ? column(std::integral_constant<int, BM>(), wm0 + i * 16 + r16) + kq * BM * (int)sizeof(double) : 0;
#pragma unroll
  for (int j = 0; j < TN; ++j) b_col[j] = BM * 128 + column(std::integral_constant<int, BN>(), wn0 + j * 16 + r16) + kq * BN * (int)sizeof(double);

  const int chain = CHAINS ? (int)(P.k_chain / BK) : nkt;
  for (int kt0 = 0; kt0 < nkt; kt0 += chain) {
    const int kt1 = CHAINS && kt0 + chain < nkt ? kt0 + chain : nkt;
    for (int kt = kt0; kt < kt1; ++kt) {
      // tile kt has landed once at most the loads of the S - 2 tiles behind it are outstanding
      asm volatile("" ::: "memory");
      if (kt + S - 1 <= nkt) __builtin_amdgcn_s_waitcnt(pipe_wait((S - 2) * LOADS));
      else __builtin_amdgcn_s_waitcnt(pipe_wait(0));
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      const char *st = pipe_lds + (kt % S) * STAGE;
      if (kt + 1 == nkt && last_k < BK) {
        // (of both operands: an infinity among what was read would make a NaN of zeros on one side)
        char *at = pipe_lds + (kt % S) * STAGE;
        PipeLoad<BM, TA>::clear(at, last_k, tid);
        PipeLoad<BN, true>::clear(at + BM * 128, last_k, tid);
        __syncthreads();
      }
      issue();
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        double af[TM][V], bf[V][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          if (TA) {
#pragma unroll
            for (int e = 0; e < V; ++e)
              af[i][e] = *reinterpret_cast<const double *>(st + (4 * V * t + 4 * e) * BM * (int)sizeof(double) + a_col[i]);
          } else {
            const piece_t x = *reinterpret_cast<const piece_t *>(st + a_row[i] + (((4 * t + kq) ^ a_swz) << 4));
#pragma unroll
            for (int e = 0; e < V; ++e) af[i][e] = x[e];
          }
        }
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            bf[e][j] = *reinterpret_cast<const double *>(st + (4 * V * t + 4 * e) * BN * (int)sizeof(double) + b_col[j]);
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = Mfma<double>::run(af[i][e], bf[e][j], acc[i][j]);
      }
    }
    if constexpr (CHAINS) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          sum[i][j] += acc[i][j];
          acc[i][j] = (f64x4)0.0;
        }
    }
  }
  if constexpr (CHAINS) gemm_epilogue<double, double, double, TM, TN, EPI>(P, sum, split, m0 + wm0, n0 + wn0, lane);
  else gemm_epilogue<double, double, double, TM, TN, EPI>(P, acc, split, m0 + wm0, n0 + wn0, lane);
}

// ---------------------------------------------------------------- host side

template <bool TA, int BM, int BN, int WGM, int WGN, bool CHAINS>
struct PipeRun {
  static constexpr bool kFull = !TA;      // with the full epilogue (applies, lifts) as well
  template <int EPI, bool C> static hipError_t launch(hipStream_t s, dim3 grid, const GemmParams &Q) {
    constexpr int S = pipe_stages(BM, BN, C);
    constexpr size_t lds = PipeCfg<BM, BN, S>::lds;
    hipLaunchKernelGGL((gemm_pipe_kernel<TA, BM, BN, WGM, WGN, S, EPI, C>), grid, dim3(256), lds, s, Q);
    return hipGetLastError();
  }
  static hipError_t go(hipStream_t s, const GemmParams &P, int batch) {
    GemmParams Q = P;
    Q.tiles_n = (int)ceil_div(P.N, BN);
    Q.tiles_m = (int)ceil_div(P.M, BM);
    const dim3 grid((unsigned)((int64_t)Q.tiles_n * Q.tiles_m * P.splits), (unsigned)batch);
    if (P.splits == 1 && (P.dead != nullptr || P.trans_c != 0)) {
      if constexpr (kFull) return launch<1, false>(s, grid, Q);       // (these are not cut)
      else return hipErrorInvalidValue;
    }
    return launch<0, CHAINS>(s, grid, Q);
  }
};

// What this kernel can compute: 16-byte rows, plain sums, tiles (128 rows, 128 bytes of k) of at most 4 GiB from the first to the last element.
inline bool pipe_can(const GemmDesc &d) {
  return d.lda < ((int64_t)1 << 22) && d.ldb < ((int64_t)1 << 22) && GemmDispatch<double, double, double>::aligned_a(d) && GemmDispatch<double, double, double>::aligned_b(d) && d.a_shift == nullptr && d.alpha == 1.0 && d.beta == 0.0 &&
         !(d.trans_a && (d.dead != nullptr || d.trans_c));
}

// Tiles of the result that are computed (of a symmetric one those that reach the diagonal or lie above it).
inline int64_t pipe_tiles(const GemmDesc &d, int bm, int bn) {
  const int64_t tm = ceil_div(d.M, bm), tn = ceil_div(d.N, bn);
  if (!d.upper_only) return tm * tn * d.batch;
  int64_t tiles = 0;
  for (int64_t i = 0; i < tm; ++i) tiles += tn - i * bm / bn;
  return tiles * d.batch;
}

// The number of k ranges, at most `most` (the workspace holds the partial sums of that many), that takes the least time for a product of one
// column tile.  What counts is the longest queue of a CU: its workgroups share the rate of its matrix cores, of which one alone reaches 0.55,
// four together 0.85, or its share of the memory's; 4 us for the first loads and the stores of those that run side by side; and the partial
// sums, written and read at 4.5 TB/s behind a second launch.  Over 140 products measured with up to 25 numbers of ranges each (5000 x 5000, l = 96:
// 3 125, 6 111, 7 130, 13 126 us) the one chosen is 0.4 % slower than the best (geometric mean; 5 % at most).
inline SplitChoice pipe_ranges(const rsvd_ctx *ctx, const GemmDesc &d, int bm, int bn, int64_t most) {
  constexpr int BK = kPipeBK;
  static const double share[5] = {0.0, 0.55, 0.72, 0.78, 0.85}, share_mem[5] = {0.0, 0.8, 0.9, 1.0, 1.0};
  const int64_t tiles = pipe_tiles(d, bm, bn), ktiles = ceil_div(d.K, BK), cus = ctx->cu_count;
  const int wgs = pipe_wgs(bm, bn, true);
  const double us = 2.0 * BK * bm * bn * (double)cus / 71e6, us_mem = (double)BK * bm * sizeof(double) * (double)cus / 4.8e6;      // of a k-tile
  int64_t best = 1;
  double best_cost = -1.0;
  for (int64_t r = 1; r <= most && r <= ktiles; ++r) {
    const int64_t per = ceil_div(ktiles, r), ranges = ceil_div(ktiles, per), queue = ceil_div(tiles * ranges, cus);
    const int side = (int)(queue < wgs ? queue : wgs);
    const double math = us / share[side], mem = us_mem / share_mem[side];
    const double sums = (double)ranges * (double)d.M * (double)d.N * d.batch * sizeof(double);
    const double cost = (double)(queue * per) * (math > mem ? math : mem) + 4.0 * (double)ceil_div(queue, wgs) +
                        (ranges > 1 ? 4.0 + 2.0 * sums / 4.5e6 : 0.0);
    if (best_cost < 0 || cost < best_cost) { best = r; best_cost = cost; }
  }
  SplitChoice c;
  c.k_per_split = ceil_div(ktiles, best) * BK;
  c.splits = (int)ceil_div(d.K, c.k_per_split);
  return c;
}

// by_tile: launches the kernel for this tile; chains: it can add up several chains of a range.
template <typename F>
inline hipError_t pipe_launch(rsvd_ctx *ctx, hipStream_t s, const GemmDesc &d, F by_tile) {
  if (d.batch < 1 || d.batch > 65535) return hipErrorInvalidValue;
  // The k ranges of gemm_kernel bound those taken here: the workspace is sized for their partial sums.  They are also the longest sums that go
  // into one accumulator, so that the rounding error stays that of gemm_kernel (20000 terms in one go where it has two ranges: 21 eps, not 15).
  const TileChoice t = choose_tile(d.M, d.N, d.K, sizeof(double), d.trans_a != 0, d.upper_only != 0);
  const SplitChoice was = choose_split(ctx, t, d.M, d.N, d.K, d.force_splits, d.upper_only != 0, d.batch);
  // One column tile up to 128 columns, beyond the tile with the shortest longest queue of a CU, a tile's time being its area by what
  // share of the matrix cores' rate it reached (128 rows whose workgroup is alone on its CU: less, two of 64 rows hide each other's loads).
  // Two fixed rules were slower: 128 rows and the column tile with the least padding (A^T X of 12000 x 9000, l = 200, 128 x 128 tiles 1453 us,
  // gemm_kernel 1113, now 958), and 64 x 96 everywhere (A X of 20000 x 20000, l = 288, 3886 us, now 3643; of 12000 x 9000, l = 200, 1299, now 905).
  // 70 shapes in both directions: within 0.2 % of the best tile (3.2 % at most).
  const bool chains = d.N <= 128;
  int bm = 64, bn = (int)ceil_div(d.N, 16) * 16;
  SplitChoice c = was;
  if (chains) {
    c = pipe_ranges(ctx, d, bm, bn, d.force_splits > 0 ? d.force_splits : was.splits);
  } else {
    static const struct { int bm, bn; double share; } tiles[5] = {{128, 96, 0.94}, {128, 64, 0.95}, {64, 96, 0.93}, {64, 80, 0.91}, {64, 64, 0.89}};
    double best = -1.0;
    for (const auto &t : tiles) {
      const int64_t queue = ceil_div(pipe_tiles(d, t.bm, t.bn) * was.splits, ctx->cu_count);
      const double cost = (double)(queue * t.bm * t.bn) / (queue == 1 && t.bm == 128 ? 0.8 * t.share : t.share);
      if (best < 0 || cost < best) { best = cost; bm = t.bm; bn = t.bn; }
    }
  }
  if (c.splits > 1) {
    const size_t need = (size_t)c.splits * (size_t)d.M * (size_t)d.N * sizeof(double);
    if (d.partial == nullptr || d.partial_bytes < need) return hipErrorInvalidValue;
  }
  GemmParams P = make_params(d, c, d.upper_only ? bm : 0, d.upper_only ? bn : 0);
  P.k_chain = was.k_per_split;
  hipError_t e;
  {
    ProfScope ps(ctx, s, d.prof_kind);
    e = by_tile(P, bm, bn, chains);
  }
  if (e != hipSuccess) return e;
  return finish_splits<double, double, double>(ctx, s, d, P);
}

}  // namespace rsvd
