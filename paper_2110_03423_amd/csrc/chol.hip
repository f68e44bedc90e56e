// Step 3 of Algorithm 1, small dense part: the l x l work of CholeskyQR.
//
// The paper orthonormalises the tall-skinny Y with Householder QR
// (GEQRF + ORGQR).  Here the same Q (up to column signs) comes from the Gram
// matrix: G = Y^T Y = R^T R, Q = Y R^-1, applied twice.  This file factors G
// and inverts R in fp64.  A pivot that drops below tau times the column's
// original squared norm marks the column as numerically dependent: its row of
// R and its column of R^-1 are set to zero (the caller replaces the column of
// Q by a fresh Gaussian direction), so a rank-deficient Y still gives a full
// orthonormal basis that contains range(Y).
#include "common.hpp"
#include "mfma.hpp"
#include "pivot.hpp"
#include "philox_dev.hpp"

namespace rsvd {

hipError_t gemm_launch_f64(rsvd_ctx *ctx, hipStream_t s, const GemmDesc &d);

// One workgroup of NB wavefronts factors an nb x nb block (nb <= 16 NB) and inverts the
// factor.  The block is the sum of n_parts matrices spaced part_stride elements apart
// (split-K partial Gram matrices are added here, in a fixed order).
//
// Elimination on [S | I] by 16 x 16 blocks.  Wavefront r owns block row r for the whole
// run and keeps it in registers in the accumulator layout of the fp64 matrix-core
// instruction: slot J >= r is the S block (r, J), slot J < r the block (r, J) of
// Z = R^-T.  Wavefront 0, whose own row is complete after the first step, factors all the
// diagonal blocks (diag_factor).  The chain that every
// step has to wait for is: row kb complete -> update of the next diagonal block -> its
// factorisation -> scaling of row kb + 1 by T^T, T = R_kk^-1; everything else is moved off it.
// Step kb, two barriers:
//   * row kb lies in LDS unscaled, T and R_kk are there: every other wavefront multiplies one
//     column block of the row by T^T on the matrix cores, in place (one block each instead of the
//     whole row in one wavefront); wavefront kb + 1, which has just scaled the block above its own
//     diagonal block, updates that block with it and hands it over through LDS;        -- barrier
//   * wavefront 0 factors block kb + 1 and publishes R, T and the flags, while the
//     wavefronts r > kb take  block(r, J) -= R[kb][r]^T block(kb, J)  for their (other) slots,
//     wavefront kb + 1 then leaves its row in LDS; block row kb of R and block column kb of R^-1 (the
//     transpose of Z) are written by the wavefronts whose own rows are complete, or behind their updates
//     by all but the factoring one while those are fewer than two.                     -- barrier
// What bounds it, in cycles of one factorisation (l = 77, 109): a step takes the factoring wavefront 4200 for its block and about 2000
// beside it, and the others about as long; 3400 to 4200 are the loads at the start and 1700 the stores at the end.  48100 -> 38900, 70000 -> 56400
// by a shorter elimination of the blocks (5800 -> 4200), stores that take few instructions (3500 -> 2200 of a step in each wavefront)
// and slots without work left out.  Whole calls: 10000 x 2000 fp32, l = 80, q = 2 794 -> 772 us; 2000 x 1000 fp64, l = 110, q = 2 1371 -> 1344.
//   g0    : original squared column norms for the pivot test, or NULL to use the diagonal
//   Rinv  : nb x nb block of R^-1 (ld ldri, type TOut, zeros below the diagonal)
//   R     : same for R in fp64 (ld ldr), or NULL
//   dead  : nb flags (1 = pivot <= tau * original squared norm)
template <int NB> struct CholLds {
  static constexpr int LP = 16 * NB, LD = LP + 1, TLD = 17;
  // rows of [R | Z], the inverses of the diagonal blocks, the reference norms, the diagonal block in hand
  static constexpr size_t bytes = ((size_t)LP * LD + (size_t)NB * 16 * TLD + LP + 256) * sizeof(double);
};

// Lane J of each group of sixteen to all of them.
template <int J> __device__ __forceinline__ double row_bcast(double x) {
  long v = __builtin_bit_cast(long, x);
  v = __builtin_amdgcn_update_dpp(0L, v, 0x150 + J, 0xf, 0xf, true);       // row_newbcast
  return __builtin_bit_cast(double, v);
}

// s[i] -= (t of lane i) * m for the rows I .. E - 1: one instruction a row (left to itself the compiler copies t first and adds up late,
// with every copy kept until then).  An instruction that reads other lanes needs two more between it and the one that
// wrote its operand: diag_eliminate sees to that.
template <int I, int E>
__device__ __forceinline__ void diag_rows(double (&s)[16], double t, double m) {
  if constexpr (I < E && I < 16) {
    asm volatile("v_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(s[I]) : "v"(t), "v"(m), "n"(I));
    diag_rows<I + 1, E>(s, t, m);
  }
}

// CHECK: pivots at or below their thresholds are dropped or set aside (the masks tell which).
template <int J, bool CHECK>
__device__ __forceinline__ void diag_eliminate(double (&s)[16], double t0, double m0, double thr, unsigned pos, int c, bool raise, int cols,
                                               unsigned &dmask, unsigned &wmask) {
  if constexpr (J < 16) {
    if (J % 4 == 0 && J >= cols) return;
    double d = row_bcast<J>(s[J]);                              // pivot S[J][J]
    if constexpr (CHECK) {
      const unsigned gt = (unsigned)__ballot(s[J] > thr);       // bit J: it exceeds the threshold of its column
      if ((((gt & pos) >> J) & 1u) == 0u) {
        if (raise && ((pos >> J) & 1u)) {                       // set aside: nothing of R but the raised diagonal element
          wmask |= 1u << J;
          d = row_bcast<J>(thr);
          s[J] = c == J ? d : c > J ? 0.0 : s[J];
        } else {
          dmask |= 1u << J;                                     // dependent column: a row of zeros
          d = 1.0;
          s[J] = 0.0;
        }
      }
    }
    // The row over sqrt(d): the hardware's 1 / sqrt(d) is good to ~1e-7, the series that corrects it goes to the second power of its error.
    // What is left to do with the row before, t0 and m0, stands between the steps of this chain.
    constexpr int N = J > 0 ? (15 - J + 4) / 5 : 0, R0 = J + 1;
    const double r0 = __builtin_amdgcn_rsq(d);
    diag_rows<R0, R0 + N>(s, t0, m0);
    __builtin_amdgcn_sched_barrier(0);
    const double u = s[J] * r0, w = d * r0;
    diag_rows<R0 + N, R0 + 2 * N>(s, t0, m0);
    __builtin_amdgcn_sched_barrier(0);
    const double e = fma(-w, r0, 1.0);
    diag_rows<R0 + 2 * N, R0 + 3 * N>(s, t0, m0);
    __builtin_amdgcn_sched_barrier(0);
    const double g = fma(0.375, e, 0.5), ue = u * e;
    diag_rows<R0 + 3 * N, R0 + 4 * N>(s, t0, m0);
    __builtin_amdgcn_sched_barrier(0);
    const double t = fma(ue, g, u);
    diag_rows<R0 + 4 * N, R0 + 5 * N>(s, t0, m0);
    __builtin_amdgcn_sched_barrier(0);
    const double m = c == J ? 0.0 : t;
    s[J] = t;
    if constexpr (J < 15)
      asm volatile("s_nop 1\n\tv_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf\n\ts_nop 1"
                   : "+v"(s[J + 1]) : "v"(t), "v"(m), "n"(J + 1));
    diag_eliminate<J + 1, CHECK>(s, t, m, thr, pos, c, raise, cols, dmask, wmask);
  }
}

// Factor and invert one 16 x 16 symmetric block.  One wavefront runs this alone, and every step of the elimination
// waits for the one before: the cost is the chain  pivot, one over its root, the row, the next pivot.
// Elimination on [S | I] without the second half: lane c (the four groups of sixteen lanes do the same)
// holds column c, register i row i.  With pivot j, row j is divided by sqrt(d_j) and the rows i > j take
// S[i][c] -= R[j][i] R[j][c],  those of Z = R_kk^-T the same with Z[j][c] in the place of R[j][c].  Column c of Z begins with pivot c, when
// column c of S is done with, and its entries are then -S[i][c] / d_c: kept without that factor, Z takes the place of S as it
// stands, and one fused multiply-add a row, with an element that all lanes get from lane i, does both.  The products commute, so S stays
// symmetric to the bit: Z is the inverse of this R, to the rounding of its elements, however small a pivot is (with rows scaled
// by 1 / d_j instead, of which one factor of each product has it, the two triangles drift apart by the rounding of the large elements).
// A block takes 4200 cycles (16 pivots of about 200, and its way from and to LDS); as rank-one updates by matrix instructions, 64 cycles for
// S and as many for Z, 5800.  Errors of R and R^-1 against 80-bit arithmetic, orders 16 to 128, columns over none to six decades: R^T R - G
// 0.76 to 0.99 of what they were, R^-1 R - 1 0.43 to 0.68 (with one correction of 1 / r below: 0.97 to 1.3).
//   blk  : 16 x 16 doubles in LDS, row-major: S_kk; what it holds afterwards is of no use
//   dblk, z : out, in the accumulator layout (register v of lane L: row 4 v + L / 16, column L % 16):
//          R_kk (valid on and above the diagonal), Z_kk = R_kk^-T (lower triangular)
//   thr  : lane c holds tau * (reference squared norm of column c); pos: bit c set when that norm is > 0
//          (and not below the caller's absolute floor)
//   piv  : 16 doubles of LDS scratch
//   cols : rows and columns from here on are padding, of which this makes the identity; pivots are left out four at a time.
//   raise: a pivot at or below its threshold (with a usable reference norm) does not drop its column but SETS IT
//          ASIDE: the pivot takes the value of the threshold, the row is not used to eliminate anything (its
//          part of R is the diagonal element alone), so the column comes out of Q = Y R^-1 as what is left of it
//          after the columns before it, divided by sqrt(threshold): short of unit length, with the direction it
//          still carries magnified to where the next round can resolve it, and with no large entries in R^-1
//          (eliminating with a raised pivot instead couples the weak rows by ratios far above one, and their
//          inverse overflowed on a sketch with ~100 such rows)
//   look : look at each pivot when it is due, 45 cycles a pivot more.  Otherwise they are looked at when all are done, and the
//          elimination is done again if one was too small: the caller asks for a look once there was such a pivot in its call.
//   returns the 16-bit mask of dropped (dependent) columns, and in bits 16..31 that of the columns set aside
__device__ __forceinline__ unsigned diag_factor(double *blk, f64x4 &dblk, f64x4 &z, double thr, unsigned pos, int lane,
                                                double *piv, bool raise, int cols, bool look) {
  const int lr = lane >> 4, lc = lane & 15;
  double s[16];
  auto load = [&]() {
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = blk[i <= lc ? i * 16 + lc : lc * 16 + i];       // (the upper triangle counts)
    if (cols < 16) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (i == lc && i >= cols) s[i] = 1.0;
    }
  };
  auto store = [&]() {
    if (lane < 16) {
#pragma unroll
      for (int i = 0; i < 16; ++i) blk[i * 16 + lc] = s[i];
    }
    __builtin_amdgcn_wave_barrier();
  };
  unsigned dmask = 0, wmask = 0;
  double r;                                      // R[c][c] in lane c
  auto diagonal = [&]() {
    r = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) r = i == lc ? s[i] : r;
  };
  bool done = false;
  if (!look) {
    load();
    diag_eliminate<0, false>(s, 0.0, 0.0, thr, pos, lc, raise, cols, dmask, wmask);
    diagonal();                                  // (a pivot below zero leaves NaN)
    const unsigned need = cols < 16 ? (1u << cols) - 1u : 0xffffu;
    done = ((unsigned)__ballot(pivot_surely_above(r, thr)) & pos & need) == need;
  }
  if (!done) {
    load();
    diag_eliminate<0, true>(s, 0.0, 0.0, thr, pos, lc, raise, cols, dmask, wmask);
    diagonal();
  }
  double rv = __builtin_amdgcn_rcp(r);
  rv = fma(fma(-r, rv, 1.0), rv, rv);
  rv = fma(fma(-r, rv, 1.0), rv, rv);
  rv = ((dmask >> lc) & 1u) ? 0.0 : rv;
  const double ny = ((wmask >> lc) & 1u) ? 0.0 : -rv * rv;
  store();
  if (lane < 16) piv[lc] = rv;
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int row = 4 * v + lr;
    const double x = blk[row * 16 + lc];
    dblk[v] = x;
    z[v] = lc < row ? x * ny : lc == row ? piv[row] : 0.0;
  }
  return dmask | (wmask << 16);
}

// Stores through a buffer descriptor: p plus `lane_bytes` plus `bytes` (the same for all lanes), and none for lane_bytes = kNoStore, which is
// out of the range that the descriptor states whatever `bytes` is.  The matrices here are a few MB at most.
constexpr unsigned kNoStore = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t store_buffer(void *p) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, 0x7fffffff, 0x00027000);
}
__device__ __forceinline__ void store_at(__amdgpu_buffer_rsrc_t buf, unsigned lane_bytes, unsigned bytes, double x) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), buf, lane_bytes, bytes, 0);
}
__device__ __forceinline__ void store_at(__amdgpu_buffer_rsrc_t buf, unsigned lane_bytes, unsigned bytes, float x) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), buf, lane_bytes, bytes, 0);
}

template <typename TOut, int NB>
__global__ __launch_bounds__(NB * 64) void chol_mfma_kernel(const double *__restrict__ G, int64_t ldg,
                                                                  int n_parts, int64_t part_stride, int nb,
                                                                  const double *__restrict__ g0, double tau,
                                                                  TOut *__restrict__ Rinv, int64_t ldri,
                                                                  double *__restrict__ R, int64_t ldr,
                                                                  int *__restrict__ dead, DevInfo *info,
                                                                  int64_t stride, const int *skip_flag, int raise,
                                                                  double floor_abs, double abs_thr, int *redo_skip,
                                                                  int redo_mode, double *__restrict__ Rinv_elim,
                                                                  int64_t ldre, double *__restrict__ diag_out, int diag_n) {
  typedef CholLds<NB> L;
  // redo_skip (device int, strided like the rest in a batch; may be NULL): the switch of the additional
  // CholeskyQR round that follows a factorisation with raised pivots; non-zero = that round is skipped.
  //   redo_mode 1: this launch decides alone: 0 when it raised a pivot, 1 when not (and when it is skipped itself);
  //   redo_mode 2: one of several launches of a blocked factorisation: only ever clears it.
  // Rinv_elim (fp64, ld ldre, may be NULL): a second copy of R^-1 whose columns of set-aside rows are zero.  A blocked
  // factorisation forms its panel R[j, rest] = X_jj^T G[j, rest] with it, so that the rows set aside come out zero
  // there as they do inside this kernel, and take no part in the trailing update.
  // diag_out (may be NULL): the first diag_n diagonal elements of G as they are now, for the pivot tests of the blocks behind this one.
  if (redo_skip != nullptr)
    redo_skip = reinterpret_cast<int *>(reinterpret_cast<char *>(redo_skip) + (int64_t)blockIdx.x * stride);
  if (skip_flag != nullptr &&
      *reinterpret_cast<const int *>(reinterpret_cast<const char *>(skip_flag) + (int64_t)blockIdx.x * stride) != 0) {
    if (redo_skip != nullptr && redo_mode == 1 && threadIdx.x == 0) *redo_skip = 1;
    return;
  }
  if (blockIdx.x != 0) {              // batched launch: one problem per workgroup, `stride` bytes apart
    const int64_t off = (int64_t)blockIdx.x * stride;
    G = reinterpret_cast<const double *>(reinterpret_cast<const char *>(G) + off);
    Rinv = reinterpret_cast<TOut *>(reinterpret_cast<char *>(Rinv) + off);
    if (R != nullptr) R = reinterpret_cast<double *>(reinterpret_cast<char *>(R) + off);
    dead = reinterpret_cast<int *>(reinterpret_cast<char *>(dead) + off);
  }
  if (diag_out != nullptr)
    for (int j = threadIdx.x; j < diag_n; j += NB * 64) diag_out[j] = G[(int64_t)j * ldg + j];
  constexpr int LP = L::LP, LD = L::LD, TLD = L::TLD;
  extern __shared__ double smem[];
  double *Sm = smem;                       // LP x LD: rows of [R | Z]
  double *Td = Sm + LP * LD;               // NB x 16 x TLD: R_kk^-1
  double *d0 = Td + NB * 16 * TLD;         // LP: reference squared norms for the pivot test
  double *Dg = d0 + LP;                    // 16 x 16: the diagonal block in hand
  __shared__ double piv[16];
  __shared__ int n_dead, n_weak, bad;
  __shared__ unsigned wmask_sh;            // rows of the current pivot block that were set aside
  __shared__ unsigned char aside[16 * NB];
  const int tid = threadIdx.x, lane = tid & 63;
  // Block row of this wavefront; the wavefront of row 0 also factors the diagonal blocks.  Wavefronts w and w + 4
  // share a SIMD unit and its matrix pipe: the one next to the factoring wavefront takes row 1, which is complete
  // after the first step, so that the factorisations that follow have the pipe to themselves; of two others that
  // share one, one has a low row and is done early.
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = NB > 4 ? (wv == 4 ? 1 : wv > 0 && wv < 4 ? wv + 1 : wv) : wv;
  const int lr = lane >> 4, lc = lane & 15;
  // register slot t of wavefront wr holds column block (wr + t) mod NB: slot 0 is the
  // diagonal block, slots 1 .. NB-1-wr the S blocks to its right, the rest the Z blocks
  auto col_block = [&](int t) { const int J = wr + t; return J >= NB ? J - NB : J; };

  if (tid == 0) { n_dead = 0; n_weak = 0; bad = 0; wmask_sh = 0u; }
  __syncthreads();
  // ---- load block row wr: sum of the parts for the S slots, zero for the Z slots, identity padding
  f64x4 acc[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  {
    const double *Gr = G + (int64_t)(16 * wr + lr) * ldg + 16 * wr + lc;
    for (int p = 0; p < n_parts; ++p) {
      f64x4 cur[NB];
#pragma unroll
      for (int t = 0; t < NB; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = 16 * wr + 4 * v + lr, col = 16 * (wr + t) + lc;
          cur[t][v] = (row < nb && col < nb) ? Gr[(int64_t)p * part_stride + (int64_t)(4 * v) * ldg + 16 * t] : 0.0;
        }
#pragma unroll
      for (int t = 0; t < NB; ++t) acc[t] += cur[t];
    }
    // reference norms of this row's 16 columns; unit diagonal in the padding
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = 16 * wr + 4 * v + lr;
      if (4 * v + lr != lc) continue;          // the lane that holds the diagonal element of this row
      double dv = 1.0;
      if (row < nb) dv = (g0 != nullptr) ? g0[row] : acc[0][v];
      else acc[0][v] = 1.0;
      d0[row] = dv;
      if (!(fabs(dv) <= 1.79e308)) bad = 1;      // NaN or Inf
    }
  }

  // Too small pivots are expected where the call has met some (a panel that lacks directions lacks them in every round).  The
  // counts may be those of another problem of a batch, or be changing: the result is the same with a look and without (pivot_surely_above).
  bool look = info != nullptr && (info->refilled | info->raised) != 0;
  // Wavefront 0: factor the block in Dg as diagonal block kb, publish R_kk, T = R_kk^-1 and the flags.
  auto factor_block = [&](int kb) {
    const int k0 = kb * 16;
    f64x4 dblk, z;
    const double d0c = d0[k0 + lc];
    const unsigned pos = (unsigned)__ballot(d0c > 0.0 && d0c >= floor_abs) & 0xffffu;
    // pivot threshold: tau times the column's reference norm, or the same for every column (abs_thr > 0:
    // rounds that work on a panel whose resolved columns have unit length)
    const unsigned masks = diag_factor(Dg, dblk, z, abs_thr > 0.0 ? abs_thr : tau * d0c, pos, lane, piv, raise != 0, 16, look);
    look |= masks != 0u;
    const unsigned dmask = masks & 0xffffu, wmask = masks >> 16;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = 4 * v + lr;
      Sm[(k0 + row) * LD + k0 + lc] = (lc >= row) ? dblk[v] : 0.0;          // R_kk
      Td[(k0 + lc) * TLD + row] = z[v];                                      // T[c][row] = Z[row][c]
    }
    if (lane < 16 && k0 + lane < nb) dead[k0 + lane] = (int)((dmask >> lane) & 1u);
    if (lane < 16) aside[k0 + lane] = (unsigned char)((wmask >> lane) & 1u);
    if (lane == 0) {
      const int valid = min(16, nb - k0);
      n_dead += __popc(dmask & ((1u << valid) - 1u));     // wavefront 0 is the only writer
      n_weak += __popc(wmask & ((1u << valid) - 1u));
      wmask_sh = wmask;
    }
  };
  // Row wavefront wr leaves its diagonal block in Dg and the rest of its row, unscaled, in LDS.
  auto put_diag = [&]() {
#pragma unroll
    for (int v = 0; v < 4; ++v) Dg[v * 64 + lane] = acc[0][v];
  };
  auto put_row = [&]() {
#pragma unroll
    for (int t = 1; t < NB; ++t) {
      double *dst = Sm + (16 * wr + lr) * LD + 16 * col_block(t) + lc;
#pragma unroll
      for (int v = 0; v < 4; ++v) dst[4 * v * LD] = acc[t][v];
    }
  };

  const __amdgpu_buffer_rsrc_t R_buf = store_buffer(R), X_buf = store_buffer(Rinv), E_buf = store_buffer(Rinv_elim);
  if (wr == 0) { put_diag(); put_row(); }
  __syncthreads();

#pragma unroll 1
  for (int kb = -1; kb < NB; ++kb) {                // (-1: the first diagonal block is factored)
    const int k0 = kb * 16;
    // ---- row kb times T^T, in place: wavefront J takes column block J (R to the right of the diagonal, Z to the left)
    if (kb >= 0 && wr != kb) {
      double ta[4], bo[4];
      double *blk = Sm + (k0 + lr) * LD + 16 * wr + lc;
#pragma unroll
      for (int s = 0; s < 4; ++s) { ta[s] = Td[(k0 + 4 * s + lr) * TLD + lc]; bo[s] = blk[4 * s * LD]; }
      f64x4 o = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4; ++s) o = Mfma<double>::run(ta[s], bo[s], o);
      const unsigned wmask = wmask_sh;
      if (wr > kb && wmask != 0u) {
        // rows set aside keep nothing of R to the right of the diagonal (their part of R^-1, the Z blocks, stays)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if ((wmask >> (4 * v + lr)) & 1u) o[v] = 0.0;
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) blk[4 * v * LD] = o[v];
      if (wr == kb + 1) {
        // the next pivot row brings its diagonal block up to date with the block it has just scaled (the
        // accumulator layout is the layout of both operands:  block(wr, wr) -= R[kb][wr]^T R[kb][wr])
        // and hands it over
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[0] = Mfma<double>::run(-o[s], o[s], acc[0]);
        put_diag();
      }
    }
    if (kb >= 0) __syncthreads();
    if (kb >= 0 && wr > kb) {
      // ---- trailing rows: block(wr, J) -= R[kb][wr]^T block(kb, J)
      // (slots in use: the S blocks and the Z blocks up to kb, which are the first NB - wr + kb + 1; two at a time, whose
      // matrix-core instructions do not wait for each other)
      double na[4], b[NB][4];
#pragma unroll
      for (int s = 0; s < 4; ++s) na[s] = -Sm[(k0 + 4 * s + lr) * LD + 16 * wr + lc];
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        const int J = col_block(t);
        const double *src = (J == kb) ? Td + (k0 + lc) * TLD + lr                   // Z_kk = T_kk^T
                                      : Sm + (k0 + lr) * LD + 16 * J + lc;
        const int step = (J == kb) ? 4 : 4 * LD;
#pragma unroll
        for (int s = 0; s < 4; ++s) b[t][s] = src[s * step];
      }
      const int used = NB - wr + kb + 1, first = wr == kb + 1 ? 1 : 0;           // (the diagonal block of row kb + 1 is up to date)
#pragma unroll
      for (int t = 0; t < NB; t += 2) {
        if (t >= used) break;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          if (t > 0 || first == 0) acc[t] = Mfma<double>::run(na[s], b[t][s], acc[t]);
          if (t + 1 < NB) acc[t + 1] = Mfma<double>::run(na[s], t + 1 < used ? b[t + 1][s] : 0.0, acc[t + 1]);
        }
      }
      if (first) put_row();
    } else if (wr == 0 && kb + 1 < NB) {
      factor_block(kb + 1);
    }
    // ---- block row kb of R and block column kb of R^-1 are written out (R^-1 = Z^T: column k0 + c of R^-1 is
    // row k0 + c of Z), off the critical path: by the wavefronts whose rows are complete once there are two of them, before by
    // every one but the one that factors, behind its update, and in the end by all
    const bool last = kb + 1 == NB, few = kb >= 2 && !last;
    if (kb >= 0 && (last || (wr != 0 && (!few || wr <= kb)))) {
      const int parts = last ? NB : few ? kb : NB - 1, me = last ? wr : wr - 1;
      // A wavefront takes whole rows of R, and four rows of sixteen columns of R^-1 at a time: what differs from one to the next
      // is the same for all lanes.  Instructions and branches are what this costs, so there are none for the edges: rows beyond the last
      // are the last once more, and lanes beyond it store out of the range of the buffer, where nothing happens.
      const int lds_c = min(lane, LP - 1), lds_c2 = min(64 + lane, LP - 1);
      if (R != nullptr) {
        const int rows = min(16, nb - k0);
        const unsigned off = lane < nb ? 8u * lane : kNoStore, off2 = 64 + lane < nb ? 8u * (64 + lane) : kNoStore;
        for (int i0 = me; i0 < rows; i0 += 4 * parts) {
          double v[4], v2[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int r = k0 + min(i0 + parts * u, rows - 1);
            v[u] = Sm[r * LD + lds_c];
            if (LP > 64) v2[u] = Sm[r * LD + lds_c2];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int r = k0 + min(i0 + parts * u, rows - 1);
            store_at(R_buf, off, 8u * (unsigned)(r * (int)ldr), lane >= r ? v[u] : 0.0);
            if (LP > 64) store_at(R_buf, off2, 8u * (unsigned)(r * (int)ldr), 64 + lane >= r ? v2[u] : 0.0);
          }
        }
      }
      const int c = k0 + lc, groups = (nb + 3) / 4;
      const bool cleared = Rinv_elim != nullptr && aside[c];
      const unsigned off = (unsigned)sizeof(TOut) * (unsigned)(lr * (int)ldri + c), off_e = 8u * (unsigned)(lr * (int)ldre + c);
      for (int g0 = me; g0 < groups; g0 += 4 * parts) {
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int r0 = 4 * min(g0 + parts * u, groups - 1);
          const double *src = r0 >= k0 ? Td + r0 * TLD + lr * TLD + lc : Sm + c * LD + r0 + lr;
          v[u] = *src;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int r0 = 4 * min(g0 + parts * u, groups - 1);
          const bool in = r0 + lr < nb && c < nb;
          const double x = r0 + lr <= c ? v[u] : 0.0;
          store_at(X_buf, in ? off : kNoStore, (unsigned)sizeof(TOut) * (unsigned)(r0 * (int)ldri), (TOut)x);
          if (Rinv_elim != nullptr) store_at(E_buf, in ? off_e : kNoStore, 8u * (unsigned)(r0 * (int)ldre), cleared ? 0.0 : x);
        }
      }
    }
    if (!last) __syncthreads();
  }
  if (tid == 0) {                          // (the counts are this wavefront's own)
    if (info != nullptr) {
      if (n_dead > 0) atomicAdd(&info->refilled, n_dead);
      if (n_weak > 0) atomicAdd(&info->raised, n_weak);
      if (bad) atomicMax(&info->status, (int)RSVD_ERR_NONFINITE);
    }
    if (redo_skip != nullptr) {
      if (redo_mode == 1) *redo_skip = (n_weak > 0) ? 0 : 1;
      else if (n_weak > 0) *redo_skip = 0;
    }
  }
}

// ---------------------------------------------------------------- small fp32 panels: every round in one workgroup
//
// A panel of up to 16 columns that fits in LDS: all CholeskyQR rounds of a call (Gram matrix, factor and inverse, apply, the
// product of the triangular factors) in one workgroup, the panel in LDS from the first to the last.  As separate
// kernels a round is three or four launches of 3 to 8 us that wait for each other.  What bounds it is the chain of pivots in
// one wavefront (diag_factor).  Arithmetic and rules are those of the separate kernels: Gram matrix and factor in fp64, R^-1
// rounded to fp32, the apply in fp32.  Singular values of a 300 x 200 matrix, l = 16, one power iteration: 148 -> 117 us.
// (Tried for 17 to 32 columns, where the second pivot block doubles the chain: 700 x 500, l = 32, 293 -> 347 us; for fp64
// panels, whose matrix instructions and replacement columns are too much for one CU: 512 x 256, l = 20, 506 -> 535 us.)
struct PanelParams {
  int rows, l, ldy;
  const float *src; int64_t ld_src;
  float *dst; int64_t ld_dst;
  int rounds;
  double tau;
  uint64_t seed; uint32_t refill_stream; double refill_scale;
  float *Rinv; double *R1;                // R^-1 of the last round, R of the first (NULL: not wanted), ld l
  double *Rout;                           // product of all factors, ld l, or NULL
  DevInfo *info;
  const int *skip_flag;
};
constexpr int kPanelThreads = 512;        // (1024: the factoring wavefront has half the registers and its chain spills, 2x slower)
constexpr int kPanelMat = 16 * 17;
constexpr size_t kPanelFixed = (8 * 256 + 256 + 16 + 3 * kPanelMat) * sizeof(double);

// Replacement columns of a panel in LDS.  A group of the generator holds four consecutive elements of the panel: with many columns to
// replace the threads share out the groups, those of the same four columns to the lanes of a wavefront where l allows it, and
// pairs that nobody wants are left out; with few columns they share out the elements.  1024 x 16, two rounds: fifteen columns replaced
// 132 us element by element, now 80; eight 96, now 74; separate kernels 83 to 99 and 84 to 95 on three machines.  What is left is
// the generator's arithmetic on one CU, which the separate kernels spread over many.  So calls with panels of 1000 rows, l = 16 and most columns to replace take longer
// than with separate kernels: 1024 x 1024, two power iterations, rank 1 takes 314 us (separate kernels 261), rank 3 326 (274), rank 7
// 320 (285), rank 9 319 (299); rank 14 297 (346) and full rank 233 (271) less.  A call of its own, or its registers cost the
// factorisation some of theirs.
__device__ __attribute__((noinline)) void panel_refill(float *Y, int rows, int l, int ldy, unsigned dead, double scale,
                                                       uint32_t stream, uint64_t seed) {
  const int nf = __popc(dead);
  const bool groups = 4 * nf >= l, by_columns = l % 4 == 0;      // by_columns: a wavefront stays with the same four columns
  const int count = groups ? (rows * l + 3) / 4 : rows * nf;
  for (int i = threadIdx.x; i < count; i += kPanelThreads) {
    int r, c, only = -1;                             // first element of the group; the one that is asked for, or all of them
    if (!groups) {
      r = i / nf;
      unsigned left = dead;
      for (int n = i - r * nf; n > 0; --n) left &= left - 1u;
      const int e = r * l + __ffs(left) - 1;
      only = e & 3;
      r = (e & ~3) / l;
      c = (e & ~3) - r * l;
    } else if (by_columns) {
      c = i / rows;
      r = i - c * rows;
      c *= 4;
    } else {
      r = 4 * i / l;
      c = 4 * i - r * l;
    }
    const uint64_t g = (uint64_t)((r * l + c) >> 2);
    int at[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool take = r < rows && (only < 0 ? ((dead >> c) & 1u) != 0u : only == u);
      at[u] = take ? r * ldy + c : -1;
      if (++c == l) { c = 0; ++r; }
    }
    const bool first = at[0] >= 0 || at[1] >= 0, second = at[2] >= 0 || at[3] >= 0;
    if (!first && !second) continue;
    const Philox4 p = philox4x32_10(g, stream, seed);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h == 0 ? first : second) {
        double z0, z1;
        box_muller(uniform24(p.x[2 * h]), uniform24(p.x[2 * h + 1]), z0, z1);
        if (at[2 * h] >= 0) Y[at[2 * h]] = (float)(scale * z0);
        if (at[2 * h + 1] >= 0) Y[at[2 * h + 1]] = (float)(scale * z1);
      }
    }
  }
}

__global__ __launch_bounds__(kPanelThreads) void panel_qr_kernel(const PanelParams P) {
  constexpr int LD = 17, NT = kPanelThreads;
  if (P.skip_flag != nullptr && *P.skip_flag != 0) return;
  extern __shared__ double smem[];
  double *part = smem;                           // [wavefront][256]
  double *Gt = part + 8 * 256;                   // the Gram matrix
  double *piv = Gt + 256;
  double *Rl = piv + 16, *Ra = Rl + kPanelMat;   // the factor of this round, the product so far
  float *Xl = reinterpret_cast<float *>(Ra + kPanelMat);                        // R^-1
  float *Y = reinterpret_cast<float *>(smem + kPanelFixed / sizeof(double));    // [rows16][ldy]
  __shared__ unsigned dead_sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane >> 4, lc = lane & 15;
  const int rows = P.rows, l = P.l, ldy = P.ldy, rows16 = (rows + 15) & ~15;

  for (int e0 = tid; e0 < rows16 * l; e0 += 8 * NT) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = e0 + NT * u, r = e / l, c = e - r * l;
      v[u] = r < rows ? P.src[(int64_t)r * P.ld_src + c] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = e0 + NT * u, r = e / l, c = e - r * l;
      if (r < rows16) Y[r * ldy + c] = v[u];
    }
  }
  int refilled = 0, bad = 0;
  bool look = P.info != nullptr && P.info->refilled != 0;
  for (int round = 0; round < P.rounds; ++round) {
    __syncthreads();
    // ---- Gram matrix: the wavefronts share the rows
    {
      f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      const float *y = Y + lr * ldy + (lc < l ? lc : 0);
      for (int s0 = wave; s0 < rows16 / 4; s0 += 4 * 8) {
        double a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int s = s0 + u * 8;
          a[u] = (s < rows16 / 4 && lc < l) ? (double)y[4 * s * ldy] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = Mfma<double>::run(a[u], a[u], acc);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) part[wave * 256 + (4 * v + lr) * 16 + lc] = acc[v];
    }
    __syncthreads();
    if (tid < 256) {
      double sum = part[tid];
#pragma unroll
      for (int w = 1; w < 8; ++w) sum += part[w * 256 + tid];
      Gt[tid] = sum;
    }
    __syncthreads();
    // ---- factor and inverse (wavefront 0); the padding of the Gram matrix is the identity
    if (wave == 0) {
      f64x4 d, z;
      const double d0 = lc < l ? Gt[lc * 17] : 1.0;
      if (__ballot(!(fabs(d0) <= 1.79e308))) bad = 1;
      const unsigned pos = (unsigned)__ballot(d0 > 0.0) & 0xffffu;
      const unsigned dead = diag_factor(Gt, d, z, P.tau * d0, pos, lane, piv, false, l, look) & ((1u << l) - 1u);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = 4 * v + lr;
        Rl[row * LD + lc] = lc >= row ? d[v] : 0.0;
        Xl[lc * LD + row] = lc <= row ? (float)z[v] : 0.f;       // R^-1 = Z^T
      }
      refilled += __popc(dead);
      look |= dead != 0u;
      if (lane == 0) dead_sh = dead;
    }
    __syncthreads();
    const unsigned dead = dead_sh;
    // ---- the factors that the caller wants
    if (tid < l * l) {
      const int i = tid / l, j = tid - i * l;
      if (P.Rinv != nullptr) P.Rinv[tid] = Xl[i * LD + j];
      if (P.R1 != nullptr && round == 0) P.R1[tid] = Rl[i * LD + j];
    }
    if (P.Rout != nullptr) {
      // Ra <- Rl Ra, row sums in ascending order
      const int i = tid >> 4, j = tid & 15;
      double acc = 0.0;
      if (tid < 256) {
        if (round == 0) acc = Rl[i * LD + j];
        else
          for (int t = i; t <= j; ++t) acc = fma(Rl[i * LD + t], Ra[t * LD + j], acc);
      }
      __syncthreads();
      if (tid < 256) Ra[i * LD + j] = acc;
    }
    // ---- apply: a wavefront takes 16 rows at a time; they are its own, so the result replaces them
    float b[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) b[s] = Xl[(4 * s + lr) * LD + lc];
    for (int t = wave; t < rows16 / 16; t += NT / 64) {
      const float *row = Y + (16 * t + lc) * ldy;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      float a[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) a[s] = (4 * s + lr < l) ? row[4 * s + lr] : 0.f;
#pragma unroll
      for (int s = 0; s < 4; ++s) acc = Mfma<float>::run(a[s], b[s], acc);
      if (lc < l) {
#pragma unroll
        for (int v = 0; v < 4; ++v) Y[(16 * t + Mfma<float>::row(lane, v)) * ldy + lc] = acc[v];
      }
    }
    if (dead != 0u) {
      __syncthreads();
      panel_refill(Y, rows, l, ldy, dead, P.refill_scale, P.refill_stream + (uint32_t)round, P.seed);
    }
  }
  __syncthreads();
  for (int e = tid; e < rows * l; e += NT) {
    const int r = e / l, c = e - r * l;
    P.dst[(int64_t)r * P.ld_dst + c] = Y[r * ldy + c];
  }
  if (P.Rout != nullptr && tid < l * l) P.Rout[tid] = Ra[(tid / l) * LD + tid % l];
  if (tid == 0 && P.info != nullptr) {
    if (refilled > 0) atomicAdd(&P.info->refilled, refilled);
    if (bad) atomicMax(&P.info->status, (int)RSVD_ERR_NONFINITE);
  }
}

// Columns of a panel row in LDS, and what the whole takes.
static int panel_ld(int64_t l) { return (int)align_up((size_t)l, 2) + 4; }
static size_t panel_lds_bytes(int64_t rows, int64_t l) {
  return kPanelFixed + align_up((size_t)rows, 16) * panel_ld(l) * sizeof(float);
}

// One fp32 problem (the workgroups of a batch fill the chip as separate kernels) of up to 16 columns and 1024 rows: a
// 600 x 600 call with l = 8 takes 208 -> 178 us; with the panel of 1500 rows here as well, a 1500 x 300 one with l = 16 is no
// faster than without (237, 218 us).
bool panel_qr_takes(rsvd_dtype dtype, int64_t rows, int64_t l, int batch) {
  return dtype == RSVD_F32 && batch == 1 && l <= 16 && rows <= 1024;
}

hipError_t panel_qr_launch(rsvd_ctx *ctx, hipStream_t s, const PanelQr &q) {
  PanelParams P;
  P.rows = (int)q.rows; P.l = (int)q.l; P.ldy = panel_ld(q.l);
  P.src = q.src; P.ld_src = q.ld_src; P.dst = q.dst; P.ld_dst = q.ld_dst;
  P.rounds = q.rounds; P.tau = q.tau;
  P.seed = q.seed; P.refill_stream = q.refill_stream; P.refill_scale = 1.0 / sqrt((double)q.rows);
  P.Rinv = q.Rinv; P.R1 = q.R1; P.Rout = q.Rout; P.info = q.info; P.skip_flag = q.skip_flag;
  ProfScope ps(ctx, s, PK_CHOL);
  hipLaunchKernelGGL(panel_qr_kernel, dim3(1), dim3(kPanelThreads), panel_lds_bytes(q.rows, q.l), s, P);
  return hipGetLastError();
}

template <typename TOut>
__global__ void convert_matrix_kernel(const double *__restrict__ src, int64_t n_elems, TOut *__restrict__ dst,
                                      const int *skip_flag) {
  if (skip_flag != nullptr && *skip_flag != 0) return;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_elems;
       e += (int64_t)gridDim.x * blockDim.x)
    dst[e] = (TOut)src[e];
}

__global__ void fill_zero_f64_kernel(double *__restrict__ p, int64_t n, const int *skip_flag) {
  if (skip_flag != nullptr && *skip_flag != 0) return;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    p[e] = 0.0;
}

// out = R2 R1, then R3 out, then R4 out (those whose switch is not NULL and reads 0) for upper triangular fp64 matrices, l x l, ld l.
// The columns of the product are independent of each other: a workgroup takes sixteen through the whole chain.  A row of the
// product wants the rows from its own on, so groups of kChainRows rows are done from the top, in place, a group in registers
// before the first of it is stored.  What bounds it is the trip to L2 per 32 columns of R, which the row blocks of a wavefront share.
// One launch where every factor had one of its own and a copy (an element per thread; one product 54 us at l = 576, 8 at 80, now 50 and 5).  With the strip kernel above writing its results in their final type and the
// first block keeping the diagonal (four to five launches less per blocked factorisation, 4 to 5 us each, skipped or not): 4001 x 50021 fp32, l = 210, q = 1
// 4522 -> 4452 us; 20000 x 20000 fp64, l = 288, q = 2 27997 -> 27716.
constexpr int kChainBlocks = 5, kChainRows = 16 * 8 * kChainBlocks;
__global__ __launch_bounds__(512) void r_chain_kernel(int l, const double *R1, const double *R2, const double *R3, const double *R4,
                                                      double *out, int64_t stride, const int *skip3, const int *skip4) {
  const int64_t off = (int64_t)blockIdx.y * stride;        // batched: bytes between problems
  auto at = [&](const double *p) { return reinterpret_cast<const double *>(reinterpret_cast<const char *>(p) + off); };
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), r16 = lane & 15, kq = lane >> 4;
  const int c0 = (int)blockIdx.x * 16, col = c0 + r16, ccol = min(col, l - 1);
  const int lp = (l + 15) & ~15, kend = min(c0 + 16, lp);  // below kend these columns are zero
  double *dst = reinterpret_cast<double *>(reinterpret_cast<char *>(out) + off);
  typedef double pair_t __attribute__((ext_vector_type(2), aligned(8)));
  const int last = max(l - 2, 0);                          // where the last pair of a row begins (l = 1: the element behind is padding)
  for (int f = 0; f < 3; ++f) {
    const double *R = f == 0 ? R2 : f == 1 ? R3 : R4;
    if (f > 0) {
      const int *skip = f == 1 ? skip3 : skip4;
      if (skip == nullptr || *reinterpret_cast<const int *>(reinterpret_cast<const char *>(skip) + off) != 0) continue;
    }
    R = at(R);
    const double *S = f == 0 ? at(R1) : dst;
    for (int g0 = 0; g0 < lp; g0 += kChainRows) {
      f64x4 acc[kChainBlocks];
#pragma unroll
      for (int n = 0; n < kChainBlocks; ++n) acc[n] = f64x4{0.0, 0.0, 0.0, 0.0};
      for (int k0 = g0 + 16 * wave; k0 < kend; k0 += 32) {
        pair_t a[kChainBlocks][4];
        double b[4][2];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int e = 0; e < 2; ++e) b[u][e] = S[(int64_t)min(k0 + 8 * u + 2 * kq + e, l - 1) * l + ccol];
        // (64 bytes of a row per instruction, no row blocks that begin behind these columns: 50 us at l = 576, 17 at 288; 32 bytes and all blocks: 144, 45)
#pragma unroll
        for (int n = 0; n < kChainBlocks; ++n) {
          const int row = g0 + 16 * (wave + 8 * n);
          if (row >= k0 + 32 || row >= kend) break;
#pragma unroll
          for (int u = 0; u < 4; ++u)
            a[n][u] = *reinterpret_cast<const pair_t *>(R + (int64_t)min(row + r16, l - 1) * l + min(k0 + 8 * u + 2 * kq, last));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < kChainBlocks; ++n) {
          const int row = g0 + 16 * (wave + 8 * n);
          if (row >= k0 + 32 || row >= kend) break;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int k = k0 + 8 * u + 2 * kq;
            const double a0 = k <= last ? a[n][u][0] : a[n][u][1], a1 = a[n][u][1];
            acc[n] = Mfma<double>::run(k >= row + r16 && k < l ? a0 : 0.0, k <= col ? b[u][0] : 0.0, acc[n]);
            acc[n] = Mfma<double>::run(k + 1 >= row + r16 && k + 1 < l ? a1 : 0.0, k + 1 <= col ? b[u][1] : 0.0, acc[n]);
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int n = 0; n < kChainBlocks; ++n)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = g0 + 16 * (wave + 8 * n) + Mfma<double>::row(lane, v);
          if (row < l && col < l) dst[(int64_t)row * l + col] = row <= col ? acc[n][v] : 0.0;
        }
      __threadfence_block();
      __syncthreads();
    }
  }
}

__global__ void zero_ints_kernel(int *p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

int chol_max_block(const rsvd_ctx *ctx) {
  (void)ctx;
  return 128;      // 8 x 8 blocks of 16 x 16 in 149 KB of LDS
}

size_t chol_scratch_elems(const rsvd_ctx *ctx, int64_t l) {
  if (l <= chol_max_block(ctx)) return 0;
  // blocked path: g0 (l, padded to even) + fp64 R^-1 (l*l) + R (l*l) + product scratch (l*l) + the inverse of one
  // diagonal block with the columns of set-aside rows cleared (128 x 128)
  return (size_t)l + 1 + 3 * (size_t)l * (size_t)l + 128 * 128;
}

template <typename TOut>
static hipError_t launch_block(hipStream_t s, const double *G, int64_t ldg, int n_parts, int64_t part_stride, int nb,
                               const double *g0, double tau, TOut *Rinv, int64_t ldri, double *R, int64_t ldr,
                               int *dead, DevInfo *info, int batch, int64_t stride, const int *skip_flag,
                               const CholPivoting &pv, int redo_mode, double *Rinv_elim = nullptr,
                               int64_t ldre = 0, double *diag_out = nullptr, int diag_n = 0) {
  // one workgroup, one wavefront per 16-row block
#define RSVD_CHOL_CASE(NBV)                                                                                         \
  hipLaunchKernelGGL((chol_mfma_kernel<TOut, NBV>), dim3(batch), dim3(NBV * 64), CholLds<NBV>::bytes, s, G,         \
                     ldg, n_parts, part_stride, nb, g0, tau, Rinv, ldri, R, ldr, dead, info, stride, skip_flag,     \
                     pv.raise, pv.floor_abs, pv.abs_thr, pv.redo_skip, redo_mode, Rinv_elim, ldre,      \
                     diag_out, diag_n)
  switch ((nb + 15) / 16) {
    case 1: RSVD_CHOL_CASE(1); break;
    case 2: RSVD_CHOL_CASE(2); break;
    case 3: RSVD_CHOL_CASE(3); break;
    case 4: RSVD_CHOL_CASE(4); break;
    case 5: RSVD_CHOL_CASE(5); break;
    case 6: RSVD_CHOL_CASE(6); break;
    case 7: RSVD_CHOL_CASE(7); break;
    case 8: RSVD_CHOL_CASE(8); break;
    default: return hipErrorInvalidValue;
  }
#undef RSVD_CHOL_CASE
  return hipGetLastError();
}

// The kernels of this file that need more LDS than the default limit of a launch (64 KB): raised once per context.
template <typename TOut>
static hipError_t chol_raise_lds_limits() {
  hipError_t e = hipSuccess;
#define RSVD_CHOL_ATTR(NBV)                                                                              \
  if (e == hipSuccess && CholLds<NBV>::bytes > 60 * 1024)                                                \
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&chol_mfma_kernel<TOut, NBV>),                \
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)CholLds<NBV>::bytes)
  RSVD_CHOL_ATTR(1); RSVD_CHOL_ATTR(2); RSVD_CHOL_ATTR(3); RSVD_CHOL_ATTR(4);
  RSVD_CHOL_ATTR(5); RSVD_CHOL_ATTR(6); RSVD_CHOL_ATTR(7); RSVD_CHOL_ATTR(8);
#undef RSVD_CHOL_ATTR
  return e;
}

// Blocks of X = R^-1 above the diagonal blocks, given R (upper triangular, l x l) and the inverted diagonal
// blocks X_jj (nb x nb, nb = 16 * NW) already in place in X.  Column c of X depends on nothing but R and the
// X_ii: block row i of a column is  X_i = -X_ii (R[i, i+1 ..] X[i+1 .., c]),  from the diagonal block upwards.  So
// one workgroup takes a strip of 16 columns through the whole back substitution with the strip in LDS, every
// strip at once - one launch where a blocked forward scheme needs two small products per block column, each
// waiting for the one before.  Wavefront w owns rows 16 w .. 16 w + 15 of the block row in hand.
//   LDS: the strip ((rows up to the end of its diagonal block) x 17), one block row of products (nb x 17) and
//   a chunk of R (nb x 34).
// The strip goes to Xout as float or double, and that of R to Rout if it is wanted, both with zeros below the diagonal (l x l, ld l).
template <int NW>
__global__ __launch_bounds__(64 * NW) void tri_inverse_strip_kernel(const double *__restrict__ R,
                                                                    const double *__restrict__ X, int l,
                                                                    void *Xout, int out_f32, double *__restrict__ Rout,
                                                                    const int *skip_flag) {
  if (skip_flag != nullptr && *skip_flag != 0) return;
  constexpr int nb = 16 * NW, LDS_ = 17;
  const int c0 = (int)blockIdx.x * 16;
  const int j = c0 / nb, j0 = j * nb;
  const int kend = (j0 + nb < l) ? j0 + nb : l;         // rows of the strip that the diagonal block supplies end here
  extern __shared__ double tri_smem[];
  double *Xs = tri_smem;                                // [kend][17]
  double *Ts = Xs + (size_t)kend * LDS_;                // [nb][17]
  constexpr int CK = 32, RLD = CK + 2;                  // chunk of R: nb rows x CK columns, padded rows
  constexpr int PER = (nb * (CK / 2) + 64 * NW - 1) / (64 * NW);   // pairs of elements per thread and chunk
  double *Rs = Ts + (size_t)nb * LDS_;                  // [nb][RLD]
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  for (int idx = tid; idx < (kend - j0) * 16; idx += 64 * NW) {
    const int r = j0 + idx / 16, c = idx % 16;
    Xs[r * LDS_ + c] = (c0 + c < l) ? X[(int64_t)r * l + c0 + c] : 0.0;
  }
  __syncthreads();
  for (int i = j - 1; i >= 0; --i) {
    const int i0 = i * nb;
    // operands of the second product (row 16 w + r16 of X_ii, columns 16 w ..): independent of everything this
    // kernel computes, so they travel while the first product runs
    constexpr int NX = nb / 4;
    double xv[NX];
    {
      const double *Xrow = X + (int64_t)(i0 + 16 * w + r16) * l + i0;
#pragma unroll
      for (int u = 0; u < NX; ++u) {
        const int k = 16 * w + 4 * u + kq;
        xv[u] = (k < nb) ? Xrow[k] : 0.0;
      }
    }
    // Ts = R[i0 : i0 + nb, i0 + nb : kend] Xs[i0 + nb : kend, :], the block row of R staged through LDS in
    // chunks of CK columns with coalesced loads (a lane fetching its own row of R touches sixteen cache lines
    // per instruction, and that, not the arithmetic, was the whole cost of a first version)
    {
      f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      double stage[2 * PER];
      auto fetch = [&](int kk) {
#pragma unroll
        for (int t = 0; t < PER; ++t) {
          const int e = tid + 64 * NW * t;                  // pair of columns e % (CK / 2) of row e / (CK / 2)
          const int row = e / (CK / 2), k = kk + 2 * (e % (CK / 2));
          const double *src = R + (int64_t)(i0 + row) * l + k;
          stage[2 * t] = (row < nb && k < kend) ? src[0] : 0.0;
          stage[2 * t + 1] = (row < nb && k + 1 < kend) ? src[1] : 0.0;
        }
      };
      fetch(i0 + nb);
      for (int kk = i0 + nb; kk < kend; kk += CK) {
#pragma unroll
        for (int t = 0; t < PER; ++t) {
          const int e = tid + 64 * NW * t;
          const int row = e / (CK / 2), c = 2 * (e % (CK / 2));
          if (row < nb) {
            Rs[row * RLD + c] = stage[2 * t];
            Rs[row * RLD + c + 1] = stage[2 * t + 1];
          }
        }
        __syncthreads();
        if (kk + CK < kend) fetch(kk + CK);
#pragma unroll
        for (int u = 0; u < CK / 4; ++u) {
          const int k = kk + 4 * u + kq;
          const double bv = (k < kend) ? Xs[k * LDS_ + r16] : 0.0;
          acc = Mfma<double>::run(Rs[(16 * w + r16) * RLD + 4 * u + kq], bv, acc);
        }
        __syncthreads();
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) Ts[(16 * w + Mfma<double>::row(lane, v)) * LDS_ + r16] = acc[v];
    }
    __syncthreads();
    // Xs[i0 : i0 + nb, :] = -X_ii Ts   (X_ii is upper triangular: columns from this row block on; its operands
    // were fetched before the product above)
    {
      f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int u = 0; u < NX; ++u) {
        const int k = 16 * w + 4 * u + kq;
        const double bv = (k < nb) ? Ts[k * LDS_ + r16] : 0.0;
        acc = Mfma<double>::run(xv[u], bv, acc);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) Xs[(i0 + 16 * w + Mfma<double>::row(lane, v)) * LDS_ + r16] = -acc[v];
    }
    __syncthreads();
  }
  for (int idx = tid; idx < l * 16; idx += 64 * NW) {
    const int r = idx / 16, c = idx % 16;
    if (c0 + c >= l) continue;
    const int64_t at = (int64_t)r * l + c0 + c;
    const double x = r < kend ? Xs[r * LDS_ + c] : 0.0;
    if (out_f32) reinterpret_cast<float *>(Xout)[at] = (float)x;
    else reinterpret_cast<double *>(Xout)[at] = x;
    if (Rout != nullptr) Rout[at] = r <= c0 + c ? R[at] : 0.0;
  }
}

hipError_t chol_init_device(rsvd_ctx *ctx) {
  (void)ctx;
  hipError_t e = chol_raise_lds_limits<float>();
  if (e == hipSuccess) e = chol_raise_lds_limits<double>();
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&panel_qr_kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)panel_lds_bytes(1024, 16));
  const void *const strips[3] = {reinterpret_cast<const void *>(&tri_inverse_strip_kernel<6>),
                                 reinterpret_cast<const void *>(&tri_inverse_strip_kernel<7>),
                                 reinterpret_cast<const void *>(&tri_inverse_strip_kernel<8>)};
  for (const void *k : strips)
    if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 4096);
  return e;
}

static size_t tri_strip_lds(int64_t l, int nb) { return ((size_t)(l + nb) * 17 + (size_t)nb * 34) * sizeof(double); }

// Block of the blocked factorisation: 96, or wider and even where that makes a block less (a block costs a factorisation, a panel and a
// trailing update that wait for each other): l = 210 as 112 + 98 and not 96 + 96 + 18.  Whole calls with six factorisations: 4001 x 50021 fp32,
// l = 210, q = 1 4576 -> 4468 us; 8000 x 2000 fp64, q = 1, l = 211 3306 -> 3187, 310 4765 -> 4693, 380 5927 -> 5804.
static int chol_block(const rsvd_ctx *ctx, int64_t l) {
  const int64_t blocks = ceil_div(l, 128);
  const int nb = (int)ceil_div(l, 16 * blocks) * 16;
  return blocks < ceil_div(l, 96) && tri_strip_lds(l, nb) + 4096 <= (size_t)ctx->lds_per_block ? nb : 96;
}

hipError_t chol_inverse_launch(rsvd_ctx *ctx, hipStream_t s, rsvd_dtype out_dtype, int64_t l, double *G,
                               int64_t ldg, int n_parts, int64_t part_stride, double tau, void *Rinv, double *R,
                               int *dead, DevInfo *info, double *scratch, int batch, int64_t stride,
                               const int *skip_flag, const CholPivoting &pv) {
  const int nbmax = chol_max_block(ctx);
  if (batch < 1 || batch > 65535) return hipErrorInvalidValue;
  if (l <= nbmax) {
    ProfScope ps(ctx, s, PK_CHOL);
    if (out_dtype == RSVD_F32)
      return launch_block<float>(s, G, ldg, n_parts, part_stride, (int)l, nullptr, tau, (float *)Rinv, l, R, l, dead,
                                 info, batch, stride, skip_flag, pv, 1);
    return launch_block<double>(s, G, ldg, n_parts, part_stride, (int)l, nullptr, tau, (double *)Rinv, l, R, l, dead,
                                info, batch, stride, skip_flag, pv, 1);
  }
  if (batch != 1) return hipErrorNotSupported;       // the blocked path is not batched
  if (n_parts != 1) return hipErrorInvalidValue;     // the blocked path wants the reduced matrix

  // Blocked right-looking factorisation; diagonal blocks by the kernel above,
  // panels and trailing updates by the fp64 GEMM.  Rf/Xf hold R and R^-1 in fp64.
  // R^-1 above the diagonal blocks: one strip kernel after the factorisation when its strip fits in LDS
  // (l up to ~1000), else two products per block column inside the loop
  const size_t strip_lds = tri_strip_lds(l, chol_block(ctx, l));
  const int nb = chol_block(ctx, l);
  const bool strips = strip_lds + 4096 <= (size_t)ctx->lds_per_block;
  double *g0 = scratch;
  double *Xf = g0 + ((l + 1) & ~(int64_t)1);
  double *Rf = Xf + l * l;
  double *T = Rf + l * l;
  double *E = T + l * l;               // nb x nb (ld nb): X_jj without the columns of rows set aside
  const bool aside = pv.raise != 0;
  hipError_t e;
  if (!strips) {                       // (the strip kernel reads the blocks that are written below and nothing else)
    hipLaunchKernelGGL(fill_zero_f64_kernel, dim3(1024), dim3(256), 0, s, Xf, 2 * l * l, skip_flag);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }

  for (int64_t j0 = 0; j0 < l; j0 += nb) {
    const int64_t b = (l - j0 < nb) ? (l - j0) : nb;
    const int64_t rest = l - j0 - b;
    // diagonal block: R_jj and X_jj = R_jj^-1
    {
      ProfScope ps(ctx, s, PK_CHOL);
      // (the first one keeps the diagonal for the pivot tests of the others, before the trailing updates, and sets the switch)
      e = launch_block<double>(s, G + j0 * ldg + j0, ldg, 1, 0, (int)b, j0 > 0 ? g0 + j0 : nullptr, tau, Xf + j0 * l + j0, l,
                               Rf + j0 * l + j0, l, dead + j0, info, 1, 0, skip_flag, pv, j0 > 0 ? 2 : 1, aside ? E : nullptr, nb,
                               j0 > 0 ? nullptr : g0, (int)l);
    }
    if (e != hipSuccess) return e;
    if (rest > 0) {
      // panel: R[j, rest] = X_jj^T G[j, rest]
      GemmDesc p;
      p.trans_a = 1; p.M = b; p.N = rest; p.K = b;
      p.A = aside ? E : Xf + j0 * l + j0; p.lda = aside ? nb : l;
      p.B = G + j0 * ldg + j0 + b; p.ldb = ldg;
      p.C = Rf + j0 * l + j0 + b; p.ldc = l;
      p.force_splits = 1; p.skip_flag = skip_flag;
      if ((e = gemm_launch_f64(ctx, s, p)) != hipSuccess) return e;
      // trailing update: G[rest, rest] -= R[j, rest]^T R[j, rest]
      GemmDesc t;
      t.trans_a = 1; t.M = rest; t.N = rest; t.K = b;
      t.A = Rf + j0 * l + j0 + b; t.lda = l;
      t.B = Rf + j0 * l + j0 + b; t.ldb = l;
      t.C = G + (j0 + b) * ldg + j0 + b; t.ldc = ldg;
      t.alpha = -1.0; t.beta = 1.0; t.force_splits = 1;
      t.upper_only = 1;                 // nothing below reads the lower triangle of G
      t.skip_flag = skip_flag;
      if ((e = gemm_launch_f64(ctx, s, t)) != hipSuccess) return e;
    }
    if (j0 > 0 && !strips) {
      // inverse, block column j: X[0:j0, j] = -X[0:j0, 0:j0] (R[0:j0, j] X_jj)
      GemmDesc a;
      a.M = j0; a.N = b; a.K = b;
      a.A = Rf + j0; a.lda = l;
      a.B = Xf + j0 * l + j0; a.ldb = l;
      a.C = T; a.ldc = b; a.force_splits = 1; a.skip_flag = skip_flag;
      if ((e = gemm_launch_f64(ctx, s, a)) != hipSuccess) return e;
      GemmDesc c;
      c.M = j0; c.N = b; c.K = j0;
      c.A = Xf; c.lda = l;
      c.B = T; c.ldb = b;
      c.C = Xf + j0; c.ldc = l; c.alpha = -1.0; c.force_splits = 1; c.skip_flag = skip_flag;
      if ((e = gemm_launch_f64(ctx, s, c)) != hipSuccess) return e;
    }
  }
  if (strips) {
    ProfScope ps(ctx, s, PK_SMALL);
    const dim3 grid((unsigned)ceil_div(l, 16)), threads((unsigned)(nb * 4));
    const int f32 = out_dtype == RSVD_F32;
    if (nb == 96) hipLaunchKernelGGL((tri_inverse_strip_kernel<6>), grid, threads, strip_lds, s, Rf, Xf, (int)l, Rinv, f32, R, skip_flag);
    else if (nb == 112) hipLaunchKernelGGL((tri_inverse_strip_kernel<7>), grid, threads, strip_lds, s, Rf, Xf, (int)l, Rinv, f32, R, skip_flag);
    else hipLaunchKernelGGL((tri_inverse_strip_kernel<8>), grid, threads, strip_lds, s, Rf, Xf, (int)l, Rinv, f32, R, skip_flag);
    return hipGetLastError();
  }
  if (out_dtype == RSVD_F32) {
    hipLaunchKernelGGL((convert_matrix_kernel<float>), dim3(512), dim3(256), 0, s, Xf, l * l, (float *)Rinv, skip_flag);
  } else {
    hipLaunchKernelGGL((convert_matrix_kernel<double>), dim3(512), dim3(256), 0, s, Xf, l * l, (double *)Rinv,
                       skip_flag);
  }
  if (R != nullptr)
    hipLaunchKernelGGL((convert_matrix_kernel<double>), dim3(512), dim3(256), 0, s, Rf, l * l, R, skip_flag);
  return hipGetLastError();
}

// One workgroup per problem: sums of squares of R and of R^-1, flag = (their product <= limit^2).
template <typename T>
__global__ __launch_bounds__(1024) void cond_flag_kernel(int l, const double *__restrict__ R, const T *__restrict__ Rinv,
                                                         double limit, int *flag, DevInfo *info, int64_t stride,
                                                         const int *redo_skip) {
  const int64_t off = (int64_t)blockIdx.x * stride;
  // a factorisation with raised pivots: the panel is badly conditioned whatever the later factors look like
  const bool raised = redo_skip != nullptr &&
                      *reinterpret_cast<const int *>(reinterpret_cast<const char *>(redo_skip) + off) == 0;
  R = reinterpret_cast<const double *>(reinterpret_cast<const char *>(R) + off);
  Rinv = reinterpret_cast<const T *>(reinterpret_cast<const char *>(Rinv) + off);
  flag = reinterpret_cast<int *>(reinterpret_cast<char *>(flag) + off);
  __shared__ double part[2][16];
  __shared__ int singular;
  if (threadIdx.x == 0) singular = 0;
  __syncthreads();
  double a = 0.0, b = 0.0;
  {
    // sixteen loads in flight per thread (one after the other, l = 576 took 150 us here)
    const int nt = (int)blockDim.x, total = l * l;
    int e = threadIdx.x;
    for (; e + 7 * nt < total; e += 8 * nt) {
      double rv[8], xv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) { rv[u] = R[e + u * nt]; xv[u] = (double)Rinv[e + u * nt]; }
#pragma unroll
      for (int u = 0; u < 8; ++u) { a += rv[u] * rv[u]; b += xv[u] * xv[u]; }
    }
    for (; e < total; e += nt) {
      const double r = R[e], x = (double)Rinv[e];
      a += r * r;
      b += x * x;
    }
  }
  for (int j = threadIdx.x; j < l; j += blockDim.x)
    if (!(fabs((double)Rinv[j * l + j]) > 0.0)) singular = 1;       // a column was flagged dependent (or NaN)
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { a += __shfl_xor(a, o, 64); b += __shfl_xor(b, o, 64); }
  if ((threadIdx.x & 63) == 0) { part[0][threadIdx.x >> 6] = a; part[1][threadIdx.x >> 6] = b; }
  __syncthreads();
  if (threadIdx.x == 0) {
    a = 0.0; b = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) { a += part[0][w]; b += part[1][w]; }
    const double k2 = a * b;                     // (||R||_F ||R^-1||_F)^2 >= cond_2(R)^2
    const int f = (!raised && !singular && k2 > 0.0 && k2 <= limit * limit) ? 1 : 0;      // NaN and Inf give 0
    *flag = f;
    if (f && info != nullptr) atomicMax(&info->skipped_reorth, 1);
  }
}

hipError_t cond_flag_launch(hipStream_t s, rsvd_dtype dtype, int64_t l, const double *R, const void *Rinv,
                            double limit, int *flag, DevInfo *info, int batch, int64_t stride, const int *redo_skip) {
  if (dtype == RSVD_F32)
    hipLaunchKernelGGL(cond_flag_kernel<float>, dim3(batch), dim3(1024), 0, s, (int)l, R, (const float *)Rinv, limit,
                       flag, info, stride, redo_skip);
  else
    hipLaunchKernelGGL(cond_flag_kernel<double>, dim3(batch), dim3(1024), 0, s, (int)l, R, (const double *)Rinv, limit,
                       flag, info, stride, redo_skip);
  return hipGetLastError();
}

hipError_t r_chain_launch(hipStream_t s, int64_t l, const double *R1, const double *R2, double *out, int batch, int64_t stride,
                          const double *R3, const int *skip3, const double *R4, const int *skip4) {
  hipLaunchKernelGGL(r_chain_kernel, dim3((unsigned)ceil_div(l, 16), (unsigned)batch), dim3(512), 0, s, (int)l, R1, R2, R3, R4, out, stride,
                     skip3, skip4);
  return hipGetLastError();
}

hipError_t zero_ints_launch(hipStream_t s, int *p, int n) {
  hipLaunchKernelGGL(zero_ints_kernel, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

}  // namespace rsvd
