// fp32 products on the bf16 matrix cores, without giving up a bit of the inputs.
//
// An fp32 number is the exact sum of three bf16 numbers (x = h + m + t: 8 + 8 + 8 significand bits, each the
// rounded rest of the ones before), so  a b = sum of nine bf16 products, of which the six of order 2^-16 and above are
// taken (hh, hm, mh, mm, ht, th); what is left out, mt + tm + tt, is below 2^-24 |a b|, half a unit of the last place
// of an fp32 product (at most 1.98 2^-25 over all significands, root mean square 2^-27.5).  The products are exact in the
// matrix instruction and summed in fp32, with an eighth of the accumulation steps of the fp32 instruction: the leading
// products in one accumulator per element of C and the other five in a second, or, where the registers don't hold two (CHAIN),
// the six of a k-tile from zero and one addition.  A 16x16x32 bf16 instruction takes 16 cycles where eight 16x16x4 fp32 ones
// take 256: six of them leave a factor 2.7.  (The split of a product into bf16 parts: Henry, Tang, Heinecke, "Leveraging the
// bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", ARITH 2019.)
//
// Both operands are multiplied by 2^16 on the way in and the result by 2^-32 on the way out: the last of the three parts
// of the smallest fp32 number is then still a bf16 number (2^-149 2^16 = 2^-133), so the split is exact for every fp32 value.
// What overflows by that (results from 2^96 on, infinities, NaN) is seen in the accumulators, which stay infinite or
// undefined: a workgroup that ends so, or has got there after its first k-tile, computes its tile again with the fp32 instruction.
//
// Both operands are staged as [row][k] bf16 planes, the eight k of a matrix operand in one 16-byte chunk, so that
// matrices whose rows run along the other index are transposed by the loads of the staging (eight dwords a
// thread, one per k) and not by LDS.  The chunks of a row are XOR-swizzled with the row number, which spreads the eight
// rows a quarter-wavefront touches over all banks without padding.  Loads are unaligned-safe (a vector load of
// gfx950 needs the alignment of its element only): odd leading dimensions and odd N take the same path.
//
// Both operands are double-buffered in LDS, and everything but the matrix instructions is put in their shadow: the vector
// instructions that split the next tile of A are issued among the matrix instructions of the current one, the loads of the tile
// after it stay in flight across the barrier, and a wide B is split once (split_pack_kernel) and copied to LDS without registers.
// What bounds a wide product is then the power of the chip: at 65536 x 16384, l = 576, the matrix pipe is busy for 68 % of the cycles
// and the clock comes down to 1.6 GHz (2.0 to 2.1 under the fp32 instruction).  Narrow ones (up to 128 columns) wait for A.
// Measured against the fp32 instruction: 65536 x 16384, l = 576: A X 9.21 -> 5.81 ms, A^T X 10.04 -> 5.96 ms;
// 4001 x 50021, l = 210: 1.26 -> 0.54 and 1.27 -> 0.56 ms; 30011 x 2999, l = 61 (odd strides): 0.178 -> 0.122 and 0.206 -> 0.104 ms.
// Relative error against 64 bits at K = 16384: 2.3e-6 -> 0.8e-6.
#pragma once

#include "gemm_impl.hpp"
#include <type_traits>

namespace rsvd {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

#define RSVD_INLINE __attribute__((always_inline))

constexpr int kSplitBK = 32;                       // k-tile: one 16x16x32 instruction deep
constexpr float kSplitScale = 65536.f;             // on both operands
constexpr int kRawStride = 144;                    // bytes of an LDS row of 32 fp32 values (redo)

// Operand of s_waitcnt: at most n vector memory operations outstanding, no LDS operation.
constexpr int wait_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0070; }

// Byte offset of chunk c (eight k) of row r inside a plane of 64-byte rows.
__device__ __forceinline__ int split_chunk(int r, int c) { return r * 64 + ((c ^ ((r >> 1) & 3)) << 4); }

// Stages ROWS x 32 elements.  KROWS = false: consecutive k are consecutive in memory; true: they are `ld` apart and
// consecutive rows are consecutive.  SHIFT: an fp64 offset per column of the stored matrix (per k when KROWS is false,
// per row when it is true) is taken away, rounded once, on the way to LDS.
template <int NT, int ROWS, bool KROWS, bool SHIFT = false>
struct SplitStage {
  static constexpr int TASKS = ROWS * 4, ITERS = (TASKS + NT - 1) / NT;
  static constexpr bool WHOLE = TASKS % NT == 0;
  float x[ITERS][8];
  double sh[SHIFT ? (KROWS ? 1 : 8) : 1];

  // Row and chunk of thread `tid` in iteration `it`; threads left over in the last one repeat the first tasks (same bytes
  // to the same place) rather than branch.
  static __device__ __forceinline__ void place(int tid, int it, int &row, int &c) {
    int idx = tid + NT * it;
    if (!WHOLE && idx >= TASKS) idx = TASKS >= NT ? idx - TASKS : idx % TASKS;
    if (KROWS) { c = idx / ROWS; row = idx - c * ROWS; }
    else { row = idx >> 2; c = idx & 3; }
  }
  // The offsets of the columns this thread stages (SHIFT): of the rows once per workgroup, of the k with every tile.
  __device__ __forceinline__ void load_shift(const double *__restrict__ shift, int64_t rows_left, int64_t k_left, int tid) {
    int row, c;
    place(tid, 0, row, c);            // (the same row, or the same k, in every iteration)
    if (KROWS) sh[0] = row < rows_left ? shift[row] : 0.0;
    else {
#pragma unroll
      for (int e = 0; e < 8; ++e) sh[e] = 8 * c + e < k_left ? shift[8 * c + e] : 0.0;
    }
  }
  // Loads of iteration `it`.  Addresses are a wave-uniform base and a 32-bit byte offset per lane that does not change
  // from tile to tile (split_fits: it does not overflow).  Rows beyond the last read that one again (what comes of
  // them is not stored), k beyond the last are zero; WHOLE_K: there are none.
  template <bool WHOLE_K>
  __device__ __forceinline__ void load(int it, const float *__restrict__ origin, int64_t ld, int64_t rows_left, int64_t k_left,
                                       int tid) {
    const char *base = reinterpret_cast<const char *>(origin);
    const int last = (int)(rows_left < ROWS ? rows_left : ROWS) - 1;
    int row, c;
    place(tid, it, row, c);
    row = row < last ? row : last;
    const unsigned off = KROWS ? ((unsigned)(8 * c) * (unsigned)ld + (unsigned)row) * 4u
                               : ((unsigned)row * (unsigned)ld + (unsigned)(8 * c)) * 4u;
    if (!WHOLE_K) {
      const int kl = (int)(k_left < kSplitBK ? k_left : kSplitBK) - 1;      // (at least one k is left)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int k = 8 * c + e, kc = k < kl ? k : kl;
        const unsigned o = KROWS ? ((unsigned)kc * (unsigned)ld + (unsigned)row) * 4u
                                 : ((unsigned)row * (unsigned)ld + (unsigned)kc) * 4u;
        const float v = *reinterpret_cast<const float *>(base + o);
        x[it][e] = k <= kl ? v : 0.f;
      }
    } else if (KROWS) {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[it][e] = *reinterpret_cast<const float *>(base + (int64_t)e * ld * 4 + off);
    } else {
      const f32x4_any lo = *reinterpret_cast<const f32x4_any *>(base + off);
      const f32x4_any hi = *reinterpret_cast<const f32x4_any *>(base + 16 + off);
#pragma unroll
      for (int e = 0; e < 4; ++e) { x[it][e] = lo[e]; x[it][4 + e] = hi[e]; }
    }
  }
  // Zeros in the place of rows beyond the last.
  __device__ __forceinline__ void clear_beyond(int it, int64_t rows_left, int tid) {
    int row, c;
    place(tid, it, row, c);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[it][e] = row < rows_left ? x[it][e] : 0.f;
  }
  // Element e of iteration `it`, the offset of its column taken away.
  __device__ __forceinline__ float value(int it, int e) const {
    return SHIFT ? (float)((double)x[it][e] - sh[KROWS ? 0 : e]) : x[it][e];
  }
  // Splits iteration `it` and writes its three planes.
  __device__ __forceinline__ void store(int it, char *planes, int tid) const {
    int row, c;
    place(tid, it, row, c);
    u32x4 h, m, t;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const float a = value(it, 2 * p) * kSplitScale, b = value(it, 2 * p + 1) * kSplitScale;
      h[p] = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
      const float a1 = a - __uint_as_float(h[p] << 16), b1 = b - __uint_as_float(h[p] & 0xffff0000u);
      m[p] = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a1, b1}, bf16x2));
      const float a2 = a1 - __uint_as_float(m[p] << 16), b2 = b1 - __uint_as_float(m[p] & 0xffff0000u);
      t[p] = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a2, b2}, bf16x2));
    }
    char *dst = planes + split_chunk(row, c);
    *reinterpret_cast<u32x4 *>(dst) = h;
    *reinterpret_cast<u32x4 *>(dst + ROWS * 64) = m;
    *reinterpret_cast<u32x4 *>(dst + 2 * ROWS * 64) = t;
  }
  // Writes iteration `it` as it is, in rows of kRawStride bytes.
  __device__ __forceinline__ void store_raw(int it, char *rows, int tid) const {
    int row, c;
    place(tid, it, row, c);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = value(it, 4 * q + e);
      *reinterpret_cast<f32x4 *>(rows + row * kRawStride + c * 32 + q * 16) = v;
    }
  }
};
// Wide outputs: the column tiles of a row tile all need the same planes of B, and every row tile needs them again.
// This kernel splits B once, into the bytes a k-tile of it occupies in LDS (planes of 64-byte rows, chunks swizzled,
// zeros beyond N and K), tile after tile with the column tiles of a k-tile next to each other; the product kernel then
// copies them without touching a register.
template <int BN>
__global__ __launch_bounds__(256) void split_pack_kernel(const GemmParams P0, char *__restrict__ packed) {
  const GemmParams P = select_problem(P0);
  if (P.skip_now) return;
  const int tile_n = (int)blockIdx.x % P.tiles_n, kt = (int)blockIdx.x / P.tiles_n;
  const int64_t k0 = (int64_t)kt * kSplitBK, n0 = (int64_t)tile_n * BN;
  const int tid = threadIdx.x;
  SplitStage<256, BN, true> sb;
  char *dst = packed + (int64_t)blockIdx.x * (3 * BN * 64);
#pragma unroll
  for (int it = 0; it < sb.ITERS; ++it) {
    sb.template load<false>(it, (const float *)P.B + k0 * P.ldb + n0, P.ldb, P.N - n0, P.K - k0, tid);
    sb.clear_beyond(it, P.N - n0, tid);
    sb.store(it, dst, tid);
  }
}

// Epilogues as in gemm_kernel: 0 plain, 1 full, 3 plain with the column offsets of A taken away while staging.
// PACKED: B comes as split_pack_kernel left it.
// CHAIN: no second set of accumulators; the six terms of a k-tile are summed from zero and added to the one set there is.
// That is more vector instructions (9 % at 65536 x 16384, l = 576) but 16 registers instead of one set of accumulators, and
// outputs of one column tile of 112 or 128 columns, which split B in place and wait for A from HBM besides, are faster
// with it in A^T X (20000 x 5000, l = 120: 169 -> 155 us; 50000 x 2000, l = 112: 153 -> 145; 100000 x 1000, l = 128: 164 -> 156) and
// within 2 % of the other in A X; at 96 columns and below it is the other way round (50000 x 2000, l = 80: 133 against 140 us).
template <bool TA, int BM, int BN, int WGM, int WGN, int EPI, bool PACKED, bool CHAIN>
__global__ __launch_bounds__(64 * WGM * WGN, 2) void gemm_split_kernel(const GemmParams P0, const char *__restrict__ packed) {
  const GemmParams P = select_problem(P0);
  if (P.skip_now) return;
  constexpr int BK = kSplitBK, NT = 64 * WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 16, TN = WN / 16;
  static_assert(WM % 16 == 0 && WN % 16 == 0, "wave tile must be made of 16x16 blocks");
  constexpr bool CENTER = (EPI == 3);
  constexpr int PA = BM * 64, PB = BN * 64, BUF = 3 * (PA + PB);      // bytes of a plane, of both operands of a k-tile
  extern __shared__ __attribute__((aligned(16))) char split_lds[];
  // behind the two buffers, one int per wavefront: its accumulators have overflowed
  constexpr int WAVES = NT / 64;
  int *flags = reinterpret_cast<int *>(split_lds + 2 * BUF);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave / WGN) * WM, wn0 = (wave % WGN) * WN;
  const int r16 = lane & 15, kq = lane >> 4;
  int tile_m, tile_n, split;
  tile_of_workgroup(P, tile_m, tile_n, split);
  const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;
  const int64_t k_begin = (int64_t)split * P.k_per_split;
  int64_t k_end = (k_begin + P.k_per_split < P.K) ? (k_begin + P.k_per_split) : P.K;
  if (P.b_upper != 0 && n0 + BN < k_end) k_end = n0 + BN;      // rows of B from n0 + BN on are zero in these columns

  const float *A = (const float *)P.A;
  const float *B = (const float *)P.B;
  // The products of the leading planes and the five terms below them are summed apart: one rounding at the size of the
  // result per k-tile instead of six, and a long k range ends four to five times closer than with the fp32 instruction.
  constexpr int LN = CHAIN ? 1 : TN;
  f32x4 acc[TM][TN], low[TM][LN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = low[i][j % LN] = (f32x4)0.f;

  SplitStage<NT, BM, TA, CENTER> sa;
  SplitStage<NT, PACKED ? 16 : BN, true> sb;
  constexpr int NA = decltype(sa)::ITERS, NB = PACKED ? 0 : decltype(sb)::ITERS;
  if (CENTER && TA) sa.load_shift(P.a_shift + m0, P.M - m0, 0, tid);
  // k-tiles of this workgroup, counted from its first; all but the last are whole
  const int kt0 = (int)(k_begin / BK), nkt = k_begin < k_end ? (int)((k_end - k_begin + BK - 1) / BK) : 0;
  const int last_k = (int)(k_end - k_begin) - (nkt - 1) * BK;
  const int whole_tiles = last_k == BK ? nkt : nkt - 1;
  const float *const a_first = TA ? A + k_begin * P.lda + m0 : A + m0 * P.lda + k_begin, *a_tile = a_first;      // the next tile to be loaded
  const float *const b_first = B + k_begin * P.ldb + n0, *b_tile = b_first;
  const double *s_tile = CENTER && !TA ? P.a_shift + k_begin : nullptr;
  const int64_t a_step = TA ? BK * P.lda : BK, b_step = BK * P.ldb;
  const int m_left = (int)(P.M - m0 < BM ? P.M - m0 : BM), n_left = (int)(P.N - n0 < BN ? P.N - n0 : BN);
  // iteration w of the staging through registers: those of A, then those of B; in narrow products A X, which wait for A from
  // HBM, the other way round, so that the pieces of A have the longer time to arrive (62393 x 2646, l = 36: 184 -> 175 us, but
  // 30000 x 3000, l = 80: 135 -> 138)
  constexpr bool B_FIRST = !TA && BN <= 64;
  constexpr int FIRST_A = B_FIRST ? NB : 0, FIRST_B = B_FIRST ? 0 : NA;
  auto is_a = [](int w) RSVD_INLINE { return w >= FIRST_A && w < FIRST_A + NA; };
  auto load_part = [&](auto whole, int w, int k_left) RSVD_INLINE {
    constexpr bool W = decltype(whole)::value;
    if (is_a(w)) sa.template load<W>(w - FIRST_A, a_tile, P.lda, m_left, k_left, tid);
    else sb.template load<W>(w - FIRST_B, b_tile, P.ldb, n_left, k_left, tid);
    if (CENTER && !TA && w - FIRST_A == NA - 1) sa.load_shift(s_tile, 0, k_left, tid);     // (behind the last use of the old ones)
    if (w == NA + NB - 1) {
      a_tile += a_step;
      if (!PACKED) b_tile += b_step;
      if (CENTER && !TA) s_tile += BK;
    }
  };
  auto store_part = [&](int w, int buf) RSVD_INLINE {
    if (is_a(w)) sa.store(w - FIRST_A, split_lds + buf * BUF, tid);
    else sb.store(w - FIRST_B, split_lds + buf * BUF + 3 * PA, tid);
  };
  // PACKED: the next tile of B straight into buffer `buf`, 1024 bytes a wavefront and instruction (a wavefront without a
  // piece of its own copies the last one again: no branches)
  constexpr int PIECES = 3 * PB / 1024, ROUNDS = (PIECES + NT / 64 - 1) / (NT / 64);
  const char *b_packed = nullptr;
  int64_t b_packed_step = 0;
  if (PACKED) {
    b_packed = packed + ((int64_t)kt0 * P.tiles_n + tile_n) * (3 * PB) + lane * 16;
    b_packed_step = (int64_t)P.tiles_n * (3 * PB);
  }
  auto copy_b = [&](int buf) RSVD_INLINE {
    if constexpr (PACKED) {
      char *dst = split_lds + buf * BUF + 3 * PA;
#pragma unroll
      for (int t = 0; t < ROUNDS; ++t) {
        int piece = wave + t * (NT / 64);
        if ((t + 1) * (NT / 64) > PIECES) piece = piece < PIECES ? piece : PIECES - 1;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(b_packed + piece * 1024),
                                         (__attribute__((address_space(3))) void *)(dst + piece * 1024), 16, 0, 0);
      }
      b_packed += b_packed_step;
    }
  };
  auto load_all = [&](int k_left) RSVD_INLINE {
#pragma unroll
    for (int w = 0; w < NA + NB; ++w) load_part(std::false_type(), w, k_left);
  };
  auto store_all = [&](int buf) RSVD_INLINE {
#pragma unroll
    for (int w = 0; w < NA + NB; ++w) store_part(w, buf);
  };
  const char *ap0 = split_lds + split_chunk(wm0 + r16, kq);
  const char *bp0 = split_lds + 3 * PA + split_chunk(wn0 + r16, kq);
  // the matrix instructions of a tile; between(j) is issued among those of column block j
  auto multiply = [&](int buf, auto between) RSVD_INLINE {
    const char *ap = ap0 + buf * BUF, *bp = bp0 + buf * BUF;
    bf16x8 af[3][TM], bf[2][3];
    f32x4 sum[2][TM];
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
      for (int i = 0; i < TM; ++i) af[s][i] = *reinterpret_cast<const bf16x8 *>(ap + s * PA + i * 1024);
#pragma unroll
    for (int s = 0; s < 3; ++s) bf[0][s] = *reinterpret_cast<const bf16x8 *>(bp + s * PB);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if (j + 1 < TN) {
#pragma unroll
        for (int s = 0; s < 3; ++s) bf[(j + 1) & 1][s] = *reinterpret_cast<const bf16x8 *>(bp + s * PB + (j + 1) * 1024);
      }
      between(j);
      constexpr int order[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};      // (plane of A, plane of B)
#pragma unroll
      for (int o = 0; o < 6; ++o)
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const bf16x8 x = af[order[o][0]][i], y = bf[j & 1][order[o][1]];
          if (CHAIN) {
            sum[j & 1][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, o == 0 ? (f32x4)0.f : sum[j & 1][i], 0, 0, 0);
          } else {
            f32x4 &c = o < 5 ? low[i][j % LN] : acc[i][j];
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, c, 0, 0, 0);
          }
        }
      if (CHAIN && j > 0) {
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[i][j - 1] += sum[(j - 1) & 1][i];
      }
      __builtin_amdgcn_sched_barrier(0);       // (one column block of operands ahead, not all of them: registers)
    }
    if (CHAIN) {
#pragma unroll
      for (int i = 0; i < TM; ++i) acc[i][TN - 1] += sum[(TN - 1) & 1][i];
    }
  };

  // A barrier that leaves the last n loads in flight, which __syncthreads() would not.
  auto wait_and_meet = [&](auto n) RSVD_INLINE {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(wait_imm(decltype(n)::value));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // Whether an accumulator of the workgroup is infinite or undefined.
  auto overflowed = [&]() RSVD_INLINE {
    unsigned largest = 0u;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) largest = max(largest, __float_as_uint(acc[i][j][v]) & 0x7fffffffu);
    const bool mine = __ballot(largest >= 0x7f800000u) != 0;
    if (lane == 0) flags[wave] = mine ? 1 : 0;
    wait_and_meet(std::integral_constant<int, 63>());
    return __ballot(flags[lane & (WAVES - 1)] != 0) != 0;
  };

  int buf = 1, kt = -1;
  bool redo = false;
  const int look = whole_tiles < 24 ? -1 : 1;        // (a long range looks for overflow behind its first tile)
  if (nkt > 0) load_all(nkt > 1 ? BK : last_k);
  // On entry of an iteration tile kt lies in buffer `buf` (none before the first), the next one (if any) in the registers
  // of the stages.
  while (kt < nkt) {
    // the rule: the next tile is split and the loads of the one after it are issued among the matrix instructions
    while (kt >= 0 && kt + 2 < whole_tiles) {
      // (split first, then load: a wait for an older load while a copy to LDS is outstanding would wait for everything)
      multiply(buf, [&](int j) RSVD_INLINE {
        constexpr int LAST = NA + NB < TN ? NA + NB : TN - 1;
#pragma unroll
        for (int w = 0; w < NA + NB; ++w)
          if ((w < LAST ? w : LAST - 1) == j) store_part(w, buf ^ 1);
        if (j == LAST) {
          copy_b(buf ^ 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int w = 0; w < NA + NB; ++w) load_part(std::true_type(), w, BK);
        }
      });
      // the packed tile has landed once at most the loads of A issued behind it (8 or 2 a part) are outstanding
      wait_and_meet(std::integral_constant<int, PACKED ? (TA ? 8 : 2) * NA : 63>());
      ++kt;
      buf ^= 1;
      if (kt == look) {
        redo = overflowed();
        if (redo) kt = nkt;
      }
    }
    if (redo) break;
    if (kt + 1 < nkt) {
      copy_b(buf ^ 1);
      store_all(buf ^ 1);
      if (kt + 2 < nkt) load_all(kt + 2 < whole_tiles ? BK : last_k);
    }
    if (kt >= 0) multiply(buf, [](int) RSVD_INLINE {});
    if (PACKED) __builtin_amdgcn_s_waitcnt(wait_imm(0));
    __syncthreads();
    ++kt;
    buf ^= 1;
  }
  if (!CHAIN) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] += low[i][j % LN];
  }
  if (!redo) redo = overflowed();
  if (!redo) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] *= 1.f / (kSplitScale * kSplitScale);
  } else {
    // The whole k range with the fp32 instruction: tiles as they are in LDS, double-buffered as well; of four consecutive k that a
    // lane holds, one goes into each of four instructions.  (About what the fp32 kernel takes, see gemm_f32.hip.)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = (f32x4)0.f;
    // (the thread number anew: addresses that follow from it were worked out before the main loop otherwise, and kept)
    int tr = threadIdx.x;
    asm volatile("" : "+v"(tr));
    const int at0 = ((tr & 63) >> 4) * 16, row0 = tr & 15;
    SplitStage<NT, BM, TA, CENTER> ra;
    SplitStage<NT, BN, true> rb;
    if (CENTER && TA) ra.load_shift(P.a_shift + m0, P.M - m0, 0, tr);
    __syncthreads();                       // (the flags have been read)
    a_tile = a_first;
    b_tile = b_first;
    if (CENTER && !TA) s_tile = P.a_shift + k_begin;
    auto load_raw = [&](auto whole, int k_left) RSVD_INLINE {
      constexpr bool W = decltype(whole)::value;
#pragma unroll
      for (int w = 0; w < NA; ++w) ra.template load<W>(w, a_tile, P.lda, m_left, k_left, tr);
#pragma unroll
      for (int w = 0; w < rb.ITERS; ++w) rb.template load<W>(w, b_tile, P.ldb, n_left, k_left, tr);
      if (CENTER && !TA) { ra.load_shift(s_tile, 0, k_left, tr); s_tile += BK; }
      a_tile += a_step;
      b_tile += b_step;
    };
    auto load_next = [&](int t) RSVD_INLINE {
      if (t < whole_tiles) load_raw(std::true_type(), BK);
      else if (t < nkt) load_raw(std::false_type(), last_k);
    };
    constexpr int RAW = (BM + BN) * kRawStride, RAW_B = BM * kRawStride;
    static_assert(RAW <= BUF, "two tiles as they are take no more LDS than two split ones");
    auto store_next = [&](int t) RSVD_INLINE {
      char *raw = split_lds + (t & 1) * RAW;
#pragma unroll
      for (int w = 0; w < NA; ++w) ra.store_raw(w, raw, tr);
#pragma unroll
      for (int w = 0; w < rb.ITERS; ++w) rb.store_raw(w, raw + RAW_B, tr);
    };
    load_next(0);
    store_next(0);
    load_next(1);
#pragma unroll 1
    for (int t = 0; t < nkt; ++t) {
      const char *raw = split_lds + (t & 1) * RAW;
      __syncthreads();
      if (t + 1 < nkt) {
        store_next(t + 1);
        load_next(t + 2);
      }
#pragma unroll 1
      for (int half = 0; half < 2; ++half) {
        const int at = half * 64 + at0;
        f32x4 af[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i)
          af[i] = *reinterpret_cast<const f32x4 *>(raw + (wm0 + i * 16 + row0) * kRawStride + at);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const f32x4 bf = *reinterpret_cast<const f32x4 *>(raw + RAW_B + (wn0 + j * 16 + row0) * kRawStride + at);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < TM; ++i) acc[i][j] = Mfma<float>::run(af[i][e], bf[e], acc[i][j]);
        }
      }
    }
  }
  gemm_epilogue<float, float, float, TM, TN, EPI>(P, acc, split, m0 + wm0, n0 + wn0, lane);
}

// ---------------------------------------------------------------- host side

// Byte offsets inside a tile are 32-bit (SplitStage::load): up to 256 rows of A, 32 of B or of A^T.
inline bool split_fits(int64_t lda, int64_t ldb) { return lda < (1 << 22) && ldb < (1 << 24); }

// Column tile: one of up to 128 columns, else the fewest of at most 144, evenly filled; the same whether B is packed or not, so
// that the workgroups, their k ranges and with them every bit of the result do not depend on it.
inline int split_tile_n(int64_t N) {
  const int64_t tiles = N <= 128 ? 1 : ceil_div(N, 144);
  return (int)(ceil_div(ceil_div(N, tiles), 16) * 16);
}
// Bytes that split_pack_kernel leaves for a K x N operand.
inline size_t split_packed_bytes(int64_t K, int64_t N) {
  const int64_t bn = split_tile_n(N), tiles = ceil_div(N, bn) * ceil_div(K, kSplitBK);
  return (size_t)tiles * (size_t)(3 * bn * 64);
}
// 32 rows a wavefront, all columns of the tile.  Up to 80 columns two workgroups of four wavefronts fit in a CU beside each other
// (20000 x 5000, l = 48: 134 -> 121 us against one of eight), beyond that one of eight.
constexpr int split_tile_m(int bn) { return bn <= 80 ? 128 : 256; }
constexpr int split_wgs_per_cu(int bn) { return bn <= 80 ? 2 : 1; }
template <int BN> struct SplitTile {
  static constexpr int BM = split_tile_m(BN), WAVES = BM / 32, WGN = 1, WGM = WAVES;
  static constexpr size_t lds = (size_t)2 * 3 * 64 * (BM + BN) + WAVES * sizeof(int);      // planes, flags of the wavefronts
};

template <bool TA, int BN, bool PACKED, bool CHAIN>
hipError_t split_run(hipStream_t s, const GemmParams &P, int batch, char *packed) {
  typedef SplitTile<BN> T;
  GemmParams Q = P;
  Q.tiles_n = (int)ceil_div(P.N, BN);
  Q.tiles_m = (int)ceil_div(P.M, T::BM);
  const dim3 grid((unsigned)((int64_t)Q.tiles_n * Q.tiles_m * P.splits), (unsigned)batch);
  if (PACKED) {
    const int64_t tiles = Q.tiles_n * ceil_div(P.K, kSplitBK);
    hipLaunchKernelGGL((split_pack_kernel<BN>), dim3((unsigned)tiles), dim3(256), 0, s, Q, packed);
  }
  const bool general = P.splits == 1 && (P.dead != nullptr || P.trans_c != 0);
  if (P.a_shift != nullptr) {
    hipLaunchKernelGGL((gemm_split_kernel<TA, T::BM, BN, T::WGM, T::WGN, 3, PACKED, CHAIN>), grid, dim3(64 * T::WAVES), T::lds, s, Q, packed);
  } else if (general) {
    if constexpr (TA) return hipErrorInvalidValue;           // (takes_split: such products have op(A) = A)
    else hipLaunchKernelGGL((gemm_split_kernel<TA, T::BM, BN, T::WGM, T::WGN, 1, PACKED, CHAIN>), grid, dim3(64 * T::WAVES), T::lds, s, Q, packed);
  } else {
    hipLaunchKernelGGL((gemm_split_kernel<TA, T::BM, BN, T::WGM, T::WGN, 0, PACKED, CHAIN>), grid, dim3(64 * T::WAVES), T::lds, s, Q, packed);
  }
  return hipGetLastError();
}

#define RSVD_SPLIT_TILES_ONE(X) X(48) X(64) X(80) X(96) X(112) X(128)
#define RSVD_SPLIT_TILES(X) X(80) X(96) X(112) X(128) X(144)

template <bool TA>
hipError_t split_by_tile(hipStream_t s, const GemmParams &P, int batch, char *packed) {
  const int bn = split_tile_n(P.N);
  if (P.N <= 128) {                    // one column tile
    switch (bn) {
#define RSVD_SPLIT_CASE(BN) case BN: return split_run<TA, BN, false, (BN >= 112)>(s, P, batch, nullptr);
      RSVD_SPLIT_TILES_ONE(RSVD_SPLIT_CASE)
#undef RSVD_SPLIT_CASE
    }
  } else if (packed != nullptr) {
    switch (bn) {
#define RSVD_SPLIT_CASE(BN) case BN: return split_run<TA, BN, true, false>(s, P, batch, packed);
      RSVD_SPLIT_TILES(RSVD_SPLIT_CASE)
#undef RSVD_SPLIT_CASE
    }
  } else {                             // the same sums without the packed operand
    switch (bn) {
#define RSVD_SPLIT_CASE(BN) case BN: return split_run<TA, BN, false, false>(s, P, batch, nullptr);
      RSVD_SPLIT_TILES(RSVD_SPLIT_CASE)
#undef RSVD_SPLIT_CASE
    }
  }
  return hipErrorInvalidValue;
}
template <bool TA, int BN, int EPI, bool PACKED, bool CHAIN>
void split_raise_lds(hipError_t &e) {
  typedef SplitTile<BN> T;
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_split_kernel<TA, T::BM, BN, T::WGM, T::WGN, EPI, PACKED, CHAIN>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)T::lds);
}
template <bool TA, int BN, bool PACKED, bool CHAIN>
void split_raise_lds_all(hipError_t &e) {
  split_raise_lds<TA, BN, 0, PACKED, CHAIN>(e);
  if constexpr (!TA) split_raise_lds<TA, BN, 1, PACKED, CHAIN>(e);
  split_raise_lds<TA, BN, 3, PACKED, CHAIN>(e);
}
template <bool TA>
hipError_t split_init() {
  hipError_t e = hipSuccess;
#define RSVD_SPLIT_CASE(BN) split_raise_lds_all<TA, BN, false, (BN >= 112)>(e);
  RSVD_SPLIT_TILES_ONE(RSVD_SPLIT_CASE)
#undef RSVD_SPLIT_CASE
#define RSVD_SPLIT_CASE(BN) split_raise_lds_all<TA, BN, false, false>(e); split_raise_lds_all<TA, BN, true, false>(e);
  RSVD_SPLIT_TILES(RSVD_SPLIT_CASE)
#undef RSVD_SPLIT_CASE
  return e;
}
hipError_t split_init_n();
hipError_t split_init_t();
hipError_t split_by_tile_n(hipStream_t s, const GemmParams &P, int batch, char *packed);      // op(A) = A
hipError_t split_by_tile_t(hipStream_t s, const GemmParams &P, int batch, char *packed);      // op(A) = A^T

}  // namespace rsvd
