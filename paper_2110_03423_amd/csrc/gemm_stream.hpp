// Products C = A^T B with up to 32 (fp32) or 48 (fp64) columns, where reading A once is what takes the time.
//
// In A^T B the rows of A run along the rows of C, so the 16 bytes of a lane are V neighbouring rows of C at one k: they are the
// operands of V matrix instructions as they come from memory, and sixteen lanes read 256 bytes of a row of A.  So nothing goes through LDS
// and nothing waits at a barrier: a wavefront has 64 rows of C, D steps of four k in flight in registers, and the four wavefronts of a
// workgroup read 1024 (fp64: 2048) bytes of every row side by side.  gemm_kernel's tiles of 64 rows, dealt over the XCDs one by one, fetched A 1.9 times
// where its rows are no multiple of 128 bytes (256 x (2000 x 500) fp32, FETCH_SIZE; this kernel 1.2 times), and its 1000 workgroups write and read partial
// sums of four times as many k ranges.  Calls of rsvd_stage_gemm_atn, gemm_kernel or gemm_pipe_kernel -> this, us (reductions included):
//   fp32  9599 x 12017, l = 23  147 -> 93   78704 x 3920, l = 19  403 -> 270   8118 x 4499, l = 30  51 -> 34   14645 x 1013, l = 29  31 -> 21
//   fp64  9599 x 12017, l = 31  294 -> 183  78704 x 3920, l = 25  661 -> 471   5923 x 1303, l = 20  31 -> 21   36637 x 411, l = 27   43 -> 29
// 70 shapes of 2e5 to 5e8 entries each: 1.14 (fp32; 0.95 at 1360 x 18352, l = 12, 23 us) and 1.08 times as fast, below 20 us the same.  Of the
// batches 256 x (2000 x 500) fp32, l = 32, 281 -> 220 a product, 32 x (4000 x 1000) fp64, l = 48, 254 -> 221.  Whole calls: these batches 1511 -> 1394
// and 2219 -> 2099, 65536 x 16384 fp32, l = 16, 3133 -> 3071.
// Tried: twice the steps in flight (the batches 10 % slower, 32 columns of long products 10 % faster), the wavefronts of a workgroup on ranges of
// their own instead of taking turns (rows of A in pieces of 256 bytes: 15 % slower), the problems of a batch in the opposite order to that of the
// product before, for what the last-level cache still holds (no change).  A X, whose sixteen rows a matrix instruction takes at the same k, has pieces
// of 64 bytes a row when read like this (0.75 times as fast as gemm_kernel); through a ring of whole lines in LDS it was 0.95 times.
#pragma once

#include "gemm_impl.hpp"

namespace rsvd {

#define RSVD_GLOBAL __attribute__((address_space(1)))

constexpr int kStreamRows = 64;            // rows of C of a wavefront
constexpr int kStreamK = 4;                // k of a step
// Steps whose loads are in flight: 8 KB and more of A for each of four to eight wavefronts on a CU.
template <typename T> __host__ __device__ constexpr int stream_depth() { return sizeof(T) == 4 ? 8 : 4; }
template <typename T> constexpr int stream_max_cols() { return sizeof(T) == 4 ? 32 : 48; }
// Neighbouring columns of a lane: never more than there are.
constexpr int stream_col_blocks(int64_t N) { return (int)((N + 15) / 16); }
static_assert(stream_col_blocks(1) == 1 && stream_col_blocks(17) == 2 && stream_col_blocks(33) == 3, "N >= NB, which the kernel takes for granted");

// A lane's NB neighbouring columns of B and C (three as a structure: a vector of three takes the place of four in memory).
template <typename T, int NB> struct StreamVec { typedef T type __attribute__((ext_vector_type(NB), aligned(sizeof(T)))); };
template <typename T> struct StreamThree {
  T x[3];
  __device__ __forceinline__ T operator[](int i) const { return x[i]; }
  __device__ __forceinline__ T &operator[](int i) { return x[i]; }
};
template <typename T> struct StreamVec<T, 3> { typedef StreamThree<T> type; };

// Problem and tile of this workgroup: one XCD receives a contiguous run of both, so that the lines that neighbouring tiles of A share and
// the narrow operand of a problem are fetched into one L2.
__device__ __forceinline__ void stream_place(int &problem, int &tile) {
  const unsigned total = gridDim.x * gridDim.y, id = blockIdx.y * gridDim.x + blockIdx.x;
  const unsigned per = (total + 7) >> 3, tall = (total & 7) ? (total & 7) : 8, xcd = id & 7, local = id >> 3;
  const unsigned at = xcd < tall ? xcd * per + local : tall * per + (xcd - tall) * (per - 1) + local;
  problem = (int)(at / gridDim.x);
  tile = (int)(at - (unsigned)problem * gridDim.x);
}

// KW wavefronts of a workgroup take turns at the steps of one tile, and add their sums in LDS at the end.
// M >= V and N >= NB: what lies beyond the last row or column of C is computed as the last ones once more, and stored as the same bits.
template <typename T, int NB, int KW>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 4 : 2) void gemm_stream_kernel(const GemmParams P0) {
  int problem, tile;
  stream_place(problem, tile);
  const GemmParams P = select_problem(P0, problem);
  if (P.skip_now) return;
  constexpr int V = 16 / (int)sizeof(T), AL = 4 / V, KS = kStreamK, D = stream_depth<T>();
  typedef T vec_a __attribute__((ext_vector_type(V), aligned(sizeof(T))));
  typedef typename StreamVec<T, NB>::type vec_b;
  typedef typename Mfma<T>::vec acc_t;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kq = lane >> 4;
  const int split = tile / P.tiles_m, tile_m = tile - split * P.tiles_m;
  const int64_t m0 = ((int64_t)tile_m * (4 / KW) + wave / KW) * kStreamRows;
  if (KW == 1 && m0 >= P.M) return;
  const int64_t k_first = (int64_t)split * P.k_per_split;
  const int64_t k_end = k_first + P.k_per_split < P.K ? k_first + P.k_per_split : P.K;
  const int64_t k_begin = k_first + (wave % KW) * KS;
  const int nk = m0 < P.M && k_begin < k_end ? (int)(k_end - k_begin) : 0;
  const int groups = (nk + KS * KW * D - 1) / (KS * KW * D);

  // 32-bit offsets of the lanes from a base that the wavefront shares.  The base of a tile with fewer than V rows lies before its first
  // row, and so does what its lanes read.
  const int m_left = (int)(P.M - m0 < kStreamRows ? P.M - m0 : kStreamRows);
  const int reach = m_left < V ? m_left - V : 0;
  const int col = r16 * NB < (int)P.N - NB ? r16 * NB : (int)P.N - NB;
  auto row_of = [&](int i, int r) {                       // first of the V rows of C that lane r of load i has, from m0
    const int m = i * 16 * V + r * V;
    return m < m_left - V ? m : m_left - V;
  };
  uint32_t aoff[AL];
#pragma unroll
  for (int i = 0; i < AL; ++i)
    aoff[i] = (uint32_t)sizeof(T) * ((uint32_t)kq * (uint32_t)P.lda + (uint32_t)(row_of(i, r16) - reach));
  const uint32_t boff = (uint32_t)sizeof(T) * ((uint32_t)kq * (uint32_t)P.ldb + (uint32_t)col);
  const RSVD_GLOBAL char *Ab = (const RSVD_GLOBAL char *)((const T *)P.A + k_begin * P.lda + m0 + reach);
  const RSVD_GLOBAL char *Bb = (const RSVD_GLOBAL char *)((const T *)P.B + k_begin * P.ldb);
  const int64_t a_step = (int64_t)sizeof(T) * KW * KS * P.lda, b_step = (int64_t)sizeof(T) * KW * KS * P.ldb;

  acc_t acc[4][NB];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = (acc_t)(T)0;

  struct Step { vec_a a[AL]; vec_b b; };
  Step st[D];
  auto load_b = [&]() {
    vec_b x;
    if constexpr (NB == 3) {
#pragma unroll
      for (int j = 0; j < NB; ++j) x[j] = ((const RSVD_GLOBAL T *)(Bb + boff))[j];
    } else {
      x = *(const RSVD_GLOBAL vec_b *)(Bb + boff);
    }
    return x;
  };
  auto next = [&]() {
    Ab += a_step;
    Bb += b_step;
    // (the bases stay in scalar registers, and each step's loads behind the matrix instructions of the step they replace: moved
    // together, the first would wait for the last)
    asm volatile("" : "+s"(Ab), "+s"(Bb)::"memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto load = [&](Step &s) {
#pragma unroll
    for (int i = 0; i < AL; ++i) s.a[i] = *(const RSVD_GLOBAL vec_a *)(Ab + aoff[i]);
    s.b = load_b();
    next();
  };
  // In the last group some k do not exist: they are not read, and zero on both sides (an infinity on one would make a NaN of a zero on the
  // other).  left: k that exist, from the step's first.
  auto load_last = [&](Step &s, int left) {
    if (left >= KS) {
      load(s);
      return;
    }
    const bool there = kq < left;
#pragma unroll
    for (int i = 0; i < AL; ++i) s.a[i] = there ? *(const RSVD_GLOBAL vec_a *)(Ab + aoff[i]) : (vec_a)(T)0;
    s.b = vec_b{};
    if (there) s.b = load_b();
    next();
  };
  auto multiply = [&](const Step &s) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = Mfma<T>::run(s.a[i / V][i % V], s.b[j], acc[i][j]);
    __builtin_amdgcn_sched_barrier(0);
  };
  if (groups > 0) {
    const int last = nk - (groups - 1) * KS * KW * D;
    if (groups > 1) {
#pragma unroll
      for (int u = 0; u < D; ++u) load(st[u]);
      for (int g = 0; g < groups - 2; ++g) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
          multiply(st[u]);
          load(st[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < D; ++u) {
        multiply(st[u]);
        load_last(st[u], last - u * KS * KW);
      }
    } else {
#pragma unroll
      for (int u = 0; u < D; ++u) load_last(st[u], last - u * KS * KW);
    }
#pragma unroll
    for (int u = 0; u < D; ++u) multiply(st[u]);
  }

  T *out = P.splits > 1 ? (T *)P.partial + (int64_t)split * P.M * P.N : (T *)P.C;
  const int64_t ldo = P.splits > 1 ? P.N : P.ldc;
  auto store = [&](int i, const vec_b (&x)[4]) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      T *dst = out + (m0 + row_of(i / V, Mfma<T>::row(lane, v)) + i % V) * ldo + col;
#pragma unroll
      for (int j = 0; j < NB; ++j) dst[j] = x[v][j];
    }
  };
  if constexpr (KW == 1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      vec_b x[4];
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int j = 0; j < NB; ++j) x[v][j] = acc[i][j][v];
      store(i, x);
    }
  } else {
    // the sums of the KW wavefronts, in order; each adds and stores 4 / KW of the blocks
    __shared__ T part[4][4][4][64];          // [wavefront][block][register][lane]
    constexpr int MY = 4 / KW;
    const int w0 = wave & ~(KW - 1), i0 = (wave & (KW - 1)) * MY;
    vec_b x[MY][4];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (j > 0) __syncthreads();
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) part[wave][i][v][lane] = acc[i][j][v];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < MY; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          T sum = part[w0][i0 + i][v][lane];
#pragma unroll
          for (int w = 1; w < KW; ++w) sum += part[w0 + w][i0 + i][v][lane];
          x[i][v][j] = sum;
        }
    }
    if (m0 < P.M) {
#pragma unroll
      for (int i = 0; i < MY; ++i) store(i0 + i, x[i]);
    }
  }
}

// ---------------------------------------------------------------- host side

// Taken for plain products with A^T, from a million entries of A on (below, either kernel is a launch and a chain of loads: 735 x 657, l = 30,
// 17.6 us and 17.4).  No alignment is asked for: 16-byte loads take any address that is one of an element.
template <typename T> inline bool stream_takes(const GemmDesc &d) {
  constexpr int V = 16 / (int)sizeof(T);
  const double entries = (double)d.M * (double)d.K * (double)d.batch;
  return d.trans_a != 0 && d.N >= 1 && d.N <= stream_max_cols<T>() && d.M >= V && entries >= 1e6 && d.alpha == 1.0 && d.beta == 0.0 &&
         !d.upper_only && !d.b_upper && !d.trans_c && d.dead == nullptr && d.a_shift == nullptr && d.lda < ((int64_t)1 << 22) &&
         d.ldb < ((int64_t)1 << 22) && d.batch >= 1 && d.batch <= 65535;
}

// Wavefronts to a tile and k ranges.  What counts is the longest queue of a CU, whatever the number of wavefronts that work at it side by side
// (a 64-column piece of a row is 256 or 512 bytes of a CU's share of 5.9 TB/s; wavefronts that take turns read shorter pieces), some us for every
// workgroup of the queue, and the partial sums with their launch.  Over 92 products with up to 24 choices each (l = 6 to 48, 10^6 to 10^9 entries) the one
// taken is 0.5 % (fp32) and 1.5 % (fp64) slower than the best (geometric means; 8 % at most, 39 % at one of 19 us).  20 x 13 workgroups take 1.5 times as
// long as 20 x 12 (25536 x 4928, l = 18: 151 us; 39 x 13 of two wavefronts a tile: 104).  The ranges are never more than gemm_kernel's, for which the
// workspace has room, and no accumulator sums up more terms than there.  So wavefronts that take turns may have fewer ranges, in short products a single one, without
// a launch for the sums: gemm_kernel or gemm_pipe_kernel, with the ranges of a single wavefront, now, us: fp64 304 x 6528, l = 24 11.8, 14.0, 11.1; 240 x 4784, l = 38
// 11.9, 13.9, 10.9; 225 x 7308, l = 8 10.9, 13.7, 10.8; fp32 464 x 7280, l = 31 14.8, 13.8, 10.9.  (Beyond 12 tiles of k one range in fp64, whose matrix
// instructions take twice as long, is too long a chain: 464 x 4192, l = 36 14.5 -> 15.8, 513 x 2712, l = 47 14.6 -> 17.2.)
template <typename T>
inline int stream_ranges(const rsvd_ctx *ctx, const GemmDesc &d, SplitChoice &c) {
  const int64_t cus = ctx->cu_count, ktiles = ceil_div(d.K, 32), most = c.splits;
  const double unit = 64.0 * sizeof(T) / 23000.0;               // us for one k of 64 rows of C
  const double each = sizeof(T) == 4 ? 1.0 : 6.0;
  static const double turns[5] = {0.0, 1.0, 1.03, 0.0, 1.08};
  const bool short_k = sizeof(T) == 4 || ktiles <= 12;
  double best = -1.0;
  int best_kw = 1;
  int64_t best_s = most;
  for (int kw = 1; kw <= 4; kw *= 2) {
    const int64_t tiles = ceil_div(d.M, kStreamRows * (4 / kw)) * d.batch, least = ceil_div(most, kw);
    for (int64_t q = short_k ? -1 : 0; q <= 4; ++q) {     // q > 0: as many ranges as make queues of q; -1: as few as may be
      int64_t s = q < 0 ? least : q == 0 ? most : cus * q / tiles;
      s = s < least ? least : s > most ? most : s;
      const int64_t per = ceil_div(ktiles, s), ranges = ceil_div(ktiles, per), queue = ceil_div(tiles * ranges, cus);
      const double sums = (double)ranges * (double)d.M * (double)d.N * d.batch * sizeof(T) * 1e-6;
      const double cost = (double)(queue * per * 32 * (4 / kw)) * unit * turns[kw] + each * (double)queue + (ranges > 1 ? 6.0 + 0.9 * sums : 0.0);
      if (best < 0 || cost < best) { best = cost; best_kw = kw; best_s = s; }
    }
  }
  c.k_per_split = ceil_div(ktiles, best_s) * 32;
  c.splits = (int)ceil_div(d.K, c.k_per_split);
  return best_kw;
}

template <typename T, int NB, int KW>
inline hipError_t stream_run(hipStream_t s, const GemmParams &P, int batch) {
  GemmParams Q = P;
  Q.tiles_n = 1;
  Q.tiles_m = (int)ceil_div(P.M, kStreamRows * (4 / KW));
  const dim3 grid((unsigned)((int64_t)Q.tiles_m * P.splits), (unsigned)batch);
  hipLaunchKernelGGL((gemm_stream_kernel<T, NB, KW>), grid, dim3(256), 0, s, Q);
  return hipGetLastError();
}

template <typename T, int NB>
inline hipError_t stream_by_waves(hipStream_t s, const GemmParams &P, int kw, int batch) {
  return kw == 1 ? stream_run<T, NB, 1>(s, P, batch) : kw == 2 ? stream_run<T, NB, 2>(s, P, batch) : stream_run<T, NB, 4>(s, P, batch);
}

template <typename T>
inline hipError_t stream_launch(rsvd_ctx *ctx, hipStream_t s, const GemmDesc &d) {
  const TileChoice t = choose_tile(d.M, d.N, d.K, sizeof(T), true);
  SplitChoice c = choose_split(ctx, t, d.M, d.N, d.K, d.force_splits, false, d.batch);
  const int kw = d.force_splits > 0 ? 1 : stream_ranges<T>(ctx, d, c);
  if (c.splits > 1) {
    const size_t need = (size_t)c.splits * (size_t)d.M * (size_t)d.N * sizeof(T);
    if (d.partial == nullptr || d.partial_bytes < need) return hipErrorInvalidValue;
  }
  const GemmParams P = make_params(d, c);
  hipError_t e;
  {
    ProfScope ps(ctx, s, d.prof_kind);
    const int nb = stream_col_blocks(d.N);
    if (nb == 1) e = stream_by_waves<T, 1>(s, P, kw, d.batch);
    else if (nb == 2) e = stream_by_waves<T, 2>(s, P, kw, d.batch);
    else if constexpr (stream_col_blocks(stream_max_cols<T>()) > 2) e = stream_by_waves<T, 3>(s, P, kw, d.batch);
    else e = hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  return finish_splits<T, T, T>(ctx, s, d, P);
}

}  // namespace rsvd
