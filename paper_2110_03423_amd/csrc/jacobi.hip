// Step 5 of Algorithm 1: SVD of the small factor by one-sided Jacobi rotations.
//
// The paper's step 5 uses a Jacobi solver because up to n/2 disjoint plane
// rotations can run in parallel and a handful of sweeps suffice.  Here the
// l x l matrix M (the triangular factor of B^T) is held column-major in LDS by
// one workgroup; each sweep walks a round-robin tournament of l-1 rounds, and in
// every round the l/2 disjoint column pairs are rotated concurrently, one
// sub-wavefront group of lanes per pair.  Rotations are accumulated in J, so on
// convergence  M J = X diag(sigma)  and  M = X diag(sigma) J^T.
//
// Stopping rule (the paper gives none): a sweep in which every pair satisfies
// |a_p . a_q| <= tol * ||a_p|| * ||a_q||, tol = eps * sqrt(l); at most 60 sweeps (24 beyond the orders of the one-launch
// block kernel, where every sweep is launched in advance).  Corrections of the whole matrix, which take the place of the last sweeps,
// end by the same rule or where the one just made leaves about tol (the largest inner product before it times its angles).
// The sweep that would only confirm this is saved when the rate of the last two sweeps says what it would find
// (jacobi_done below): with rho the largest relative inner product a sweep rotated away, the next sweep meets about
// rho^2 where the method converges quadratically (the paper: "3-4 iterations ... converges quadratically"; taken for
// granted only if the last step was at least of order 1.5 and rho <= sqrt(tol) / 4), and about rho^2 / rho_prev
// where it does not - inside a cluster of nearly equal singular values the rotations are large however small the
// inner products, and a sweep gains a constant factor only; there the sweep is saved once that estimate is below
// 8 tol.  (Stopping on rho <= sqrt(tol) / 4 alone left 1e-4 (fp32) / 1e-10 (fp64) between the vectors of such a
// cluster.)
// A column whose norm has fallen below eps * ||M||_F counts as zero and is no
// longer rotated (rotating it would change its partner by less than the
// rounding level); without this floor the surplus columns of a rank-deficient M
// keep shrinking by a factor eps per sweep until they underflow.  Its singular
// value is reported as that norm and its column of X is set to zero.
#include "common.hpp"
#include "mfma.hpp"

namespace rsvd {

constexpr int kJacobiMaxSweeps = 60;      // (a loop inside the kernel: sweeps that are not needed cost nothing)

template <typename T> struct Eps;
template <> struct Eps<float>  { static constexpr float  value = 1.1920929e-07f; };
template <> struct Eps<double> { static constexpr double value = 2.220446049250313e-16; };

// Was this sweep the last one?  rho: the largest relative inner product it rotated away (0: none), rho_prev: that
// of the sweep before (negative: there was none).
__host__ __device__ __forceinline__ bool jacobi_done(float rho, float rho_prev, float tol) {
  if (rho <= tol) return true;
  if (rho_prev < 0.f) return false;                                  // one sweep says nothing about the rate
  if (rho <= 0.25f * sqrtf(tol) && rho <= rho_prev * sqrtf(rho_prev)) return true;      // next: ~rho^2 < tol
  return rho * rho <= 8.f * tol * rho_prev;                          // next: ~rho^2 / rho_prev, a few tol at most
}
// The same from the per-sweep record of the block kernels: did the sweeps up to s - 1 finish the job?
__device__ __forceinline__ bool jacobi_done_before(const int *counters, int s, float tol) {
  if (s <= 0) return false;
  return jacobi_done(__int_as_float(counters[s - 1]), s > 1 ? __int_as_float(counters[s - 2]) : -1.f, tol);
}

// DPP lane moves: no LDS traffic, unlike a shuffle.
template <int CTRL> __device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL> __device__ __forceinline__ double dpp_mov(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned int)lo);
}
// Sum over the G = 4, 8 or 16 lanes that share a column pair (16, the one in use: a whole DPP row): neighbours (quad_perm 1,0,3,2), pairs
// (quad_perm 2,3,0,1), the other quad (row_half_mirror), the other half (row_mirror).  Every lane adds the same two partial sums at each step, so all end
// with identical bits, which their rotation needs.  So the additions are kept from being fused with a product that a lane adds up (one
// alone, in fp64 up to 16 rows): each lane would add its own product unrounded and its neighbour's rounded, and turn its rows by an angle of its
// own (columns of lengths 1e-6 apart: the decomposition off by 1e-8, now by 1e-15).
template <int G, typename T> __device__ __forceinline__ T group_sum(T v) {
#pragma clang fp contract(off)
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  if (G >= 8) v += dpp_mov<0x141>(v);
  if (G == 16) v += dpp_mov<0x140>(v);
  return v;
}

template <int G> __device__ __forceinline__ float group_max(float v) {
  v = fmaxf(v, dpp_mov<0xB1>(v));
  v = fmaxf(v, dpp_mov<0x4E>(v));
  if (G >= 8) v = fmaxf(v, dpp_mov<0x141>(v));
  if (G == 16) v = fmaxf(v, dpp_mov<0x140>(v));
  return v;
}
// Sum or maximum over the wavefront.
template <bool MAX> __device__ __forceinline__ float all_lanes(float v) {
#pragma clang fp contract(off)
  v = MAX ? group_max<16>(v) : group_sum<16>(v);
#pragma unroll
  for (int m = 16; m < 64; m <<= 1) v = MAX ? fmaxf(v, __shfl_xor(v, m, 64)) : v + __shfl_xor(v, m, 64);
  return v;
}

// Reciprocal, square root and reciprocal square root from the hardware estimates
// (1 ulp in fp32; refined by Newton steps in fp64).  The rotation parameters sit
// on the serial path of every pair, so their instruction count matters.
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fast_rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double fast_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = y * (2.0 - x * y);
  y = y * (2.0 - x * y);
  return y;
}
__device__ __forceinline__ double fast_rsq(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = y * (1.5 - 0.5 * x * y * y);
  y = y * (1.5 - 0.5 * x * y * y);
  return y;
}
__device__ __forceinline__ double fast_sqrt(double x) { return x * fast_rsq(x); }

// Rotation (c, s) that orthogonalises two columns with squared norms alpha, beta
// and inner product gamma != 0:  zeta = (beta - alpha) / (2 gamma),
// t = sign(zeta) / (|zeta| + sqrt(1 + zeta^2)), c = 1 / sqrt(1 + t^2), s = c t.
template <typename T>
__device__ __forceinline__ void rotation_params(T alpha, T beta, T gamma, T &c, T &s) {
  const T zeta = (beta - alpha) * fast_rcp((T)2 * gamma);
  const T az = fabs(zeta);
  T t;
  if (az > (T)1e7) t = (T)0.5 * fast_rcp(az);                   // avoids overflow of zeta^2
  else t = fast_rcp(az + fast_sqrt((T)1 + zeta * zeta));
  t = zeta < (T)0 ? -t : t;
  c = fast_rsq((T)1 + t * t);
  s = c * t;
}

// Pair i of round r in a tournament of n2 (even) players: player n2-1 stays,
// the others rotate (circle method).  Requires r < n2 - 1 and i < n2 / 2.
__device__ __forceinline__ void tournament_pair(int n2, int r, int i, int &a, int &b) {
  const int nm1 = n2 - 1;
  if (i == 0) {
    a = nm1;
    b = r;
  } else {
    a = r + i;
    if (a >= nm1) a -= nm1;
    b = r - i;
    if (b < 0) b += nm1;
  }
}

// Pair order of the LDS-resident kernel: a recursive halving of the column set.  A set
// of columns splits into a front half A (floor) and a back half B (ceil); for |B| rounds
// column A_i meets B_{(i + r) mod |B|}, which covers every pair between A and B with all
// columns of A busy in every round; then A and B are treated the same way, side by side.
// All sets of one level have sizes that differ by at most one, so a level of sets of size
// <= ms takes ceil(ms / 2) rounds and a sweep ceil(l/2) + ceil(l/4) + ... ~ l rounds, like the
// circle method.  The point of this order: each lane group keeps its column of A in
// registers for the whole level and only the column of B travels through LDS, which halves
// the LDS traffic of a round (the LDS port, shared by the four SIMDs, is what bounds it).
struct JacLevel {
  unsigned char stat;      // column this group keeps for the level (255: none)
  unsigned char bstart;    // first column of B
  unsigned char bsize;     // |B|
  unsigned char idx;       // i: position of `stat` in A
};
constexpr int kJacLevels = 8, kJacGroups = 64;    // orders up to 128

template <typename T> using jac_unit = T __attribute__((ext_vector_type(8 / sizeof(T))));

// Columns are stored column-major with stride ldm and zero-padded to G * RPL rows.  LDS is
// accessed in 8-byte units (two floats or one double): lane lg of the group's G lanes owns
// units lg, lg + G, lg + 2 G, ... of a column (the G lanes touch one contiguous run).
template <typename T, int RPL, int G>
__device__ __forceinline__ void load_column(const T *col, int lg, jac_unit<T> (&x)[RPL / (8 / (int)sizeof(T))]) {
  const jac_unit<T> *p = reinterpret_cast<const jac_unit<T> *>(col) + lg;
#pragma unroll
  for (int r = 0; r < RPL / (8 / (int)sizeof(T)); ++r) x[r] = p[G * r];
}
template <typename T, int RPL, int G>
__device__ __forceinline__ void store_column(T *col, int lg, const jac_unit<T> (&x)[RPL / (8 / (int)sizeof(T))]) {
  jac_unit<T> *p = reinterpret_cast<jac_unit<T> *>(col) + lg;
#pragma unroll
  for (int r = 0; r < RPL / (8 / (int)sizeof(T)); ++r) p[G * r] = x[r];
}

// Rotate the pair (kept column x of M with its column u of J, in registers; column q in
// LDS).  Returns the relative size |x.y| / (|x| |y|) of the inner product it rotated away,
// 0 when it left the pair alone; turned: sum of s^2.
template <typename T, int RPL, int G>
__device__ __forceinline__ float rotate_moving(jac_unit<T> (&x)[RPL / (8 / (int)sizeof(T))],
                                               jac_unit<T> (&u)[RPL / (8 / (int)sizeof(T))], T *Mc, T *Jc, int ldm,
                                               int q, int lg, T tol, T floor2, float &turned) {
  constexpr int V = 8 / sizeof(T);          // elements per LDS access
  constexpr int NV = RPL / V;               // accesses per column per lane
  jac_unit<T> y[NV];
  load_column<T, RPL, G>(Mc + q * ldm, lg, y);
  T alpha = 0, beta = 0, gamma = 0;
#pragma unroll
  for (int r = 0; r < NV; ++r)
#pragma unroll
    for (int e = 0; e < V; ++e) {
      alpha += x[r][e] * x[r][e];
      beta += y[r][e] * y[r][e];
      gamma += x[r][e] * y[r][e];
    }
  alpha = group_sum<G>(alpha);
  beta = group_sum<G>(beta);
  gamma = group_sum<G>(gamma);
  if (alpha <= floor2 || beta <= floor2) return 0.f;
  const T rel = fabs(gamma) * fast_rsq(alpha * beta);        // |x.y| / (|x| |y|); the matrix was scaled to unit size
  if (!(rel > tol)) return 0.f;
  const float ratio = (float)rel;
  jac_unit<T> v[NV];
  load_column<T, RPL, G>(Jc + q * ldm, lg, v);
  T c, s;
  rotation_params(alpha, beta, gamma, c, s);
  turned += (float)(s * s);
#pragma unroll
  for (int r = 0; r < NV; ++r) {
    const jac_unit<T> xo = x[r];
    x[r] = c * xo - s * y[r];
    y[r] = s * xo + c * y[r];
  }
  store_column<T, RPL, G>(Mc + q * ldm, lg, y);
#pragma unroll
  for (int r = 0; r < NV; ++r) {
    const jac_unit<T> uo = u[r];
    u[r] = c * uo - s * v[r];
    v[r] = s * uo + c * v[r];
  }
  store_column<T, RPL, G>(Jc + q * ldm, lg, v);
  return ratio;
}

// Rows are padded to a whole number of 8-byte units per lane of the group (and to 16 at least).
// Column stride: the 16 lanes of a group read one contiguous run of 128 bytes, i.e. every LDS bank
// once, whatever the stride; the two extra rows only keep consecutive columns off the same phase.
__host__ __device__ inline int jacobi_rows_padded(int l, int G, int elem_size) {
  const int step = G * (8 / elem_size) > 16 ? G * (8 / elem_size) : 16;
  return ((l + step - 1) / step) * step;
}
__host__ __device__ inline int jacobi_ldm(int l, int G, int elem_size) {
  return jacobi_rows_padded(l, G, elem_size) + 2;
}

// ---- corrections of the whole matrix inside one workgroup ----
//
// What polish_kernel (further down, with the method) does with all CUs: once a sweep has left the columns close to orthogonal, all Jacobi
// angles are taken from one Gram matrix in fp64 and applied together, M <- M exp(X), J <- J exp(X).  For M and J in LDS it is a handful of
// l x l products of one CU where a sweep is l rounds that wait for each other (50 us at l = 80, a correction 15 to 25).  Last sweeps -> corrections, the whole
// decomposition, us: nearly diagonal factors l = 80 fp32 232 -> 147, 48 fp32 83 -> 62, 64 fp64 272 -> 159, 24 fp64 64 -> 49, 16 fp64 44 -> 32;
// triangular factors of Gaussian matrices l = 80 fp32 367 -> 315, 48 fp32 150 -> 134, 64 fp64 414 -> 318, 24 fp64 103 -> 88.  X and W end
// closer to orthogonal (|X^T X - I| / sqrt(l), fp32, l = 80: 18 -> 0.9 eps).
// What bounds a product: 20 dependent matrix instructions a block at l = 80 and the barrier behind them; blocks of a whole matrix are read row by row
// from LDS, those below the diagonal of symmetric ones are copies.  (As first written, 30 KB of code with registers kept in scratch memory in loops, a
// correction took 55 us at l = 80.  fp32 has none there now, fp64 keeps 3 to 24 registers of a lane in it.)
constexpr int kPolishSteps = 10;

// Largest x for a series cut behind X^2 / 2 (1), X^3 (2), X^5 (3) and X^9 (4).  The 2-norm of X is x / 1.41 if all of it is one rotation and
// about x / 2 as met behind a sweep; off orthogonality by that much: fp64 1e-15 (4: 1e-16), fp32 1e-8.  Beyond the last, X is
// halved until it is below, and E doubled as often: E <- 2 E + E E.
template <typename T> __host__ __device__ constexpr float polish_limit(int order) {
  if (sizeof(T) == 4) return order == 1 ? 2e-3f : order == 2 ? 0.02f : order == 3 ? 0.15f : 0.75f;
  return order == 1 ? 1e-5f : order == 2 ? 4e-4f : order == 3 ? 0.01f : 0.15f;
}
// Sweeps end when the angles of the last one came to this (Frobenius norm again); it is also the largest x of a correction.  A sweep
// that turned by 14 leaves 9 on triangular factors of every kind, one of 10 leaves 2 ... 6, one of 2 leaves 0.1 ... 0.35; from 9 it takes 6
// corrections, from 2 three or four.  A large x costs corrections of 80 to 100 us each (9 to 12 products), a sweep 110 us at l = 110, 170 at
// 210 and 450 at 450.
__host__ __device__ constexpr float polish_start(int l) { return l < 160 ? 4.f : l < 256 ? 7.f : 12.f; }
constexpr double kPolishFree = 0.01;        // angles up to this are taken whatever the inner product
constexpr float kPolishRate = 0.75f;        // x of a correction in units of that before; above that they do not converge

// Corrections are looked at behind a sweep whose rotations came to corr_turned (Frobenius norm of the angles), and made if those that are left come to
// kCorrStart at most and those that the correction would leave to kCorrNext.  Those are estimated from the first Gram matrix: a correction
// leaves inner products of second order, about q = x |R| / l of the lengths (x: the norm of the angles, R: the relative inner products), hence angles
// of atan(q / gap) / 2.  Where values lie in clusters the gaps are so small that these are as large as before, however small the inner
// products, and corrections do not converge (norms estimated and found next at l = 48: noise 1.6 -> 0.3, half of the values within 1e-5
// 17 -> 1).  A look costs 2 to 4 us; behind one that refused, the next is when half as much was turned.  Jacobi times in units
// of those without corrections, 24 calls of each order (8 spectra, q = 0 to 2; low rank and noise to plateaus of equal values), geometric mean and
// largest, with a norm of 5 turned, 16 wavefronts and no estimate -> now: fp32 l = 16 1.05, 1.30 -> 1.03, 1.12; 24 1.00, 1.31 -> 0.99, 1.10; 32 0.91, 1.22 ->
// 0.94, 1.11; 48 0.89, 1.20 -> 0.89, 1.03; 64 0.94, 1.26 -> 0.92, 1.11; 80 0.90, 1.19 -> 0.91, 1.07; fp64 16 1.01, 1.29 -> 0.85, 1.05; 24 0.92, 1.17 -> 0.87, 1.08;
// 32 0.81, 1.13 -> 0.80, 1.00; 48 0.81, 1.12 -> 0.79, 1.02; 64 0.86, 1.22 -> 0.83, 1.07.  (Refusing by the largest angle left, or by the largest one turned, which
// ordinary factors have as well: 0.99 to 1.01 in fp32.)
constexpr float kCorrStart = 2.f, kCorrNext = 2.f, kCorrTurnedScale = 65536.f;
__host__ __device__ constexpr float corr_turned(int l) { return l / 14.f; }
constexpr int kCorrWaves = 16;             // wavefronts that share the 16 x 16 blocks of a product, at most
// Strips into which a row of blocks of a whole matrix is cut: one for each of nb * corr_strips(nb) wavefronts, 4 nb at most.
__host__ __device__ constexpr int corr_strips(int nb) { return kCorrWaves / nb < nb ? kCorrWaves / nb : nb; }
template <typename T, int RPL> struct CorrCfg {
  static constexpr bool kFits = sizeof(T) == 4 ? RPL <= 6 : RPL <= 4;      // (M, J and two more matrices in LDS)
  static constexpr int NB = RPL <= 4 ? 1 : 2;                              // blocks of a whole matrix that a wavefront has
};
constexpr int corr_max_order(bool f32) { return f32 ? 80 : 64; }           // a wavefront has one block on or above the diagonal
// Row stride of the two matrices: four rows that are read side by side meet different banks.
__host__ __device__ inline int corr_ld(int l) {
  const int lp = (l + 15) / 16 * 16;
  return lp % 32 == 16 ? lp : lp + 16;
}

// acc[t] = sum_k p[k][0] q[k][16 t], k = 0, 4, ... steps of the matrix instruction, n4 groups of four; the operands of a group are in flight
// together.
template <typename T, int W>
__device__ __forceinline__ void corr_product(typename Mfma<T>::vec (&acc)[W], const T *p, int ldp, const T *q, int ldq, int n4) {
#pragma unroll
  for (int t = 0; t < W; ++t) acc[t] = (typename Mfma<T>::vec)(T)0;
#pragma unroll 1
  for (int n = 0; n < n4; ++n) {
    T a[4], b[4][W];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[u] = p[4 * u * ldp];
#pragma unroll
      for (int t = 0; t < W; ++t) b[u][t] = q[4 * u * ldq + 16 * t];
    }
    __builtin_amdgcn_sched_barrier(0);       // (all loads in flight before the first is waited for)
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int t = 0; t < W; ++t) acc[t] = Mfma<T>::run(a[u], b[u][t], acc[t]);
    p += 16 * ldp;
    q += 16 * ldq;
  }
}

// Tangent of the Jacobi angle, from zeta = (d_j - d_i) / (2 g): the hardware's estimates, refined once in fp64.
__device__ __forceinline__ float corr_tan(double dj, double di, double g) {
  const float z = (float)(dj - di) * fast_rcp(2.f * (float)g), az = fabsf(z);
  const float t = az > 1e7f ? 0.5f * fast_rcp(az) : fast_rcp(az + fast_sqrt(1.f + z * z));
  return z < 0.f ? -t : t;
}
__device__ __forceinline__ double once_rcp(double x) {
  const double y = __builtin_amdgcn_rcp(x);
  return y * (2.0 - x * y);
}
__device__ __forceinline__ double corr_tan64(double dj, double di, double g) {
  const double z = (dj - di) * once_rcp(2.0 * g), az = fabs(z), w = 1.0 + z * z;
  double r = __builtin_amdgcn_rsq(w);
  r = r * (1.5 - 0.5 * w * r * r);
  const double t = az > 1e7 ? 0.5 * once_rcp(az) : once_rcp(az + w * r);
  return z < 0.0 ? -t : t;
}

// Returns whether the columns of M are orthogonal now; `applied` counts the corrections.  B0, B1: ceil16(l) rows of corr_ld(l).
// The Gram matrix, X and the parts of its exponential are symmetric or antisymmetric: of those a wavefront has one block on or above the
// diagonal, whose elements stay in its registers from step to step; of whole matrices it has one or two neighbouring blocks of a row.
template <typename T, int RPL>
__device__ __forceinline__ bool lds_corrections(T *Mc, T *Jc, int ldm, T *B0, T *B1, int l, T tol, T floor2, double *nd, f32x4 *red,
                                                int &applied) {
  typedef typename Mfma<T>::vec acc_t;
  constexpr int NB = CorrCfg<T, RPL>::NB, V = 8 / (int)sizeof(T);
  const int nb = (l + 15) >> 4, ld = corr_ld(l);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // (addresses are worked out where they are used: kept in registers from step to step and through the sweeps they do not fit)
  auto lane_now = []() {
    int lane = (int)threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    return lane;
  };
  const bool has = wave < nb * (nb + 1) / 2;
  int ui = 0, uj = has ? wave : 0;
  while (uj >= nb - ui) { uj -= nb - ui; ++ui; }
  uj += ui;
  const int strips = corr_strips(nb), width = (nb + strips - 1) / strips;
  const int fi = wave % nb;
  const bool full = wave / nb < strips;
  // (the last strip of a row may be narrower: it begins further left, and its neighbour's block is computed twice)
  const int fj = (wave / nb) * width + width <= nb ? (wave / nb) * width : nb - width;
  // block (ui, uj) of sum_k P[k][i] Q[k][j]
  auto upper = [&](acc_t &m, const T *P, const T *Q) {
    const int lane = lane_now(), at = (lane >> 4) * ld + (lane & 15);
    acc_t a[1];
    if (has) corr_product<T, 1>(a, P + at + 16 * ui, ld, Q + at + 16 * uj, ld, nb);
    m = a[0];
  };
  auto each = [&](auto f) {                      // f(v, i, j)
    const int lane = lane_now();
    if (has) {
#pragma unroll
      for (int v = 0; v < 4; ++v) f(v, 16 * ui + Mfma<T>::row(lane, v), 16 * uj + (lane & 15));
    }
  };
  auto put = [&](T *B, const acc_t &m, T mirror) {       // and mirror times it on the other side of the diagonal
    each([&](int v, int i, int j) {
      B[i * ld + j] = m[v];
      if (ui != uj) B[j * ld + i] = mirror * m[v];
    });
  };
  auto strip = [&](acc_t (&m)[NB], const T *P, const T *Q, int ldq) {
    if (!full) return;
    const int lane = lane_now(), kq = lane >> 4, r16 = lane & 15;
    const T *p = P + kq * ld + r16 + 16 * fi, *q = Q + kq * ldq + r16 + 16 * fj;
    if (NB == 2 && width == 2) {
      corr_product<T, NB>(m, p, ld, q, ldq, nb);
    } else {
      acc_t a[1];
      corr_product<T, 1>(a, p, ld, q, ldq, nb);
      m[0] = a[0];
    }
  };
  auto each_full = [&](auto f) {                 // f(t, v, i, j)
    if (!full) return;
    const int lane = lane_now();
#pragma unroll
    for (int t = 0; t < NB; ++t)
      if (t < width) {
#pragma unroll
        for (int v = 0; v < 4; ++v) f(t, v, 16 * fi + Mfma<T>::row(lane, v), 16 * (fj + t) + (lane & 15));
      }
  };
  float x_before = 1e30f;
#pragma unroll 1
  for (int step = 0; step < kPolishSteps; ++step) {
    // ---- G = M^T M in fp64, its diagonal, the angles
    f64x4 g = (f64x4)0.0;
    const int lane = lane_now(), r16 = lane & 15;
    if (has) {
      const T *p = Mc + (16 * ui + r16) * ldm + V * (lane >> 4), *q = Mc + (16 * uj + r16) * ldm + V * (lane >> 4);
#pragma unroll 1
      for (int n = 0; n < nb; ++n) {
        jac_unit<T> x[4 / V], y[4 / V];
#pragma unroll
        for (int u = 0; u < 4 / V; ++u) {
          x[u] = *reinterpret_cast<const jac_unit<T> *>(p + 4 * V * u);
          y[u] = *reinterpret_cast<const jac_unit<T> *>(q + 4 * V * u);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4 / V; ++u)
#pragma unroll
          for (int e = 0; e < V; ++e) g = Mfma<double>::run((double)x[u][e], (double)y[u][e], g);
        p += 16;
        q += 16;
      }
      if (ui == uj) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (Mfma<double>::row(lane, v) == r16) nd[16 * ui + r16] = g[v];
      }
    }
    __syncthreads();
    float rho = 0.f, x2 = 0.f, open = 0.f, rel2 = 0.f;
    if (has) {
      const int j = 16 * uj + r16;
      const double dj = j < l ? nd[j] : 0.0;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 16 * ui + Mfma<double>::row(lane, v);
        const double di = i < l ? nd[i] : 0.0, gv = g[v];
        T angle = (T)0;
        if (i < j && di > (double)floor2 && dj > (double)floor2 && gv != 0.0) {
          const float rel = (float)(fabs(gv) * __builtin_amdgcn_rsq(di * dj));
          // tan of the angle as in rotation_params, then the angle itself (to the fifth order: it only has to be a good one)
          const T tn = sizeof(T) == 4 ? (T)corr_tan(dj, di, gv) : (T)corr_tan64(dj, di, gv);
          // below the threshold only where it is a small one: inside a cluster it would be large, and noise
          if (rel > (float)tol || fabs(tn) <= (T)kPolishFree) angle = tn - tn * tn * tn * ((T)(1.0 / 3.0) - (T)0.2 * tn * tn);
          const float a2 = (float)(angle * angle);
          if (rel > (float)tol) {
            rho = fmaxf(rho, rel);
            open += a2;
            rel2 += rel * rel;
          }
          x2 += a2;
        }
        if (i <= j) {
          B0[i * ld + j] = angle;
          if (i != j) B0[j * ld + i] = -angle;
        }
        __builtin_amdgcn_sched_barrier(0);             // (one angle at a time: side by side they take more registers than there are)
      }
    }
    rho = all_lanes<true>(rho);
    x2 = all_lanes<false>(x2);
    open = all_lanes<false>(open);
    rel2 = all_lanes<false>(rel2);
    if (lane == 0) red[wave] = f32x4{rho, x2, open, rel2};
    __syncthreads();
    const f32x4 sums = red[r16];
    rho = group_max<16>(sums[0]);
    x2 = group_sum<16>(sums[1]);
    open = group_sum<16>(sums[2]);
    rel2 = group_sum<16>(sums[3]);
    const float x_all = sqrtf(2.f * x2), x_now = sqrtf(2.f * open);
    if (rho <= (float)tol) return true;
    if (!(x_now <= kCorrStart) || !(x_now <= kPolishRate * x_before)) return false;
    if (step == 0) {
      // what a correction would leave, atan(y) / 2 as y / sqrt(4 + 1.62 y^2)
      const double q2 = 4.0 * (double)open * (double)rel2 / ((double)l * l);
      float next = 0.f;
      if (has) {
        const int j = 16 * uj + r16;
        const double dj = j < l ? nd[j] : 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = 16 * ui + Mfma<double>::row(lane, v);
          const double di = i < l ? nd[i] : 0.0;
          if (i < j && di > (double)floor2 && dj > (double)floor2) {
            const double t = q2 * di * dj;
            next += (float)(t * __builtin_amdgcn_rcp((dj - di) * (dj - di) + 1.62 * t));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      next = all_lanes<false>(next);
      __syncthreads();
      if (lane == 0) red[wave][0] = next;
      __syncthreads();
      if (!(2.f * group_sum<16>(red[r16][0]) <= kCorrNext * kCorrNext)) return false;
    }
    x_before = x_now;
    const int order = x_all <= polish_limit<T>(1) ? 1 : x_all <= polish_limit<T>(2) ? 2 : x_all <= polish_limit<T>(3) ? 3 : 4;
    int doublings = 0;
    for (float x = x_all; x > polish_limit<T>(4) && doublings < 7; x *= 0.5f) ++doublings;
    const T half = (T)__builtin_ldexp(1.0, -doublings);
    // ---- E = exp(half X) - I into B1 (X[i][k] = -X[k][i]; c: the symmetric part of E)
    acc_t x, c, sn, w;
    each([&](int v, int i, int j) { x[v] = B0[i * ld + j]; });
    upper(w, B0, B0);
    w *= -half * half;
    c = w * (T)0.5;
    sn = w * (T)(1.0 / 6.0);
    if (order >= 3) {
      put(B1, w, (T)1);
      __syncthreads();
      upper(w, B1, B1);
      c += w * (T)(1.0 / 24.0);
      sn += w * (T)(1.0 / 120.0);
      if (order == 4) {
        put(B0, w, (T)1);                        // (X waits in registers)
        __syncthreads();
        upper(w, B1, B0);
        c += w * (T)(1.0 / 720.0);
        sn += w * (T)(1.0 / 5040.0);
        upper(w, B0, B0);
        c += w * (T)(1.0 / 40320.0);
        sn += w * (T)(1.0 / 362880.0);
      }
      __syncthreads();
      if (order == 4) put(B0, x, (T)-1);
    }
    x *= half;
    if (order >= 2) {
      put(B1, sn, (T)1);
      __syncthreads();
      upper(w, B0, B1);
      x -= half * w;
      __syncthreads();
    }
    each([&](int v, int i, int j) {
      B1[i * ld + j] = c[v] + x[v];
      if (ui != uj) B1[j * ld + i] = c[v] - x[v];
    });
    __syncthreads();
#pragma unroll 1
    for (int d = 0; d < doublings; ++d) {              // exp(2 X) - I = 2 E + E E, the first operand read from the transpose
      acc_t e[NB];
      each_full([&](int t, int v, int i, int j) { B0[j * ld + i] = B1[i * ld + j]; });
      __syncthreads();
      strip(e, B0, B1, ld);
      each_full([&](int t, int v, int i, int j) { e[t][v] += (T)2 * B1[i * ld + j]; });
      __syncthreads();
      each_full([&](int t, int v, int i, int j) { B1[i * ld + j] = e[t][v]; });
      __syncthreads();
    }
    // ---- column i of the new M and J = that of the old one + sum_k E[k][i] column k (E is zero in the rows beyond the last column)
    {
      acc_t am[NB], aj[NB];
      strip(am, B1, Mc, ldm);
      strip(aj, B1, Jc, ldm);
      __syncthreads();
      each_full([&](int t, int v, int i, int j) {
        // (a block that two wavefronts have is stored by the one whose strip it begins in)
        if (i < l && (fj + t) / width == wave / nb) {
          Mc[i * ldm + j] += am[t][v];
          Jc[i * ldm + j] += aj[t][v];
        }
      });
      __syncthreads();
    }
    ++applied;
    if (rho * x_all <= (float)tol) return true;             // the next one would find about that
  }
  return false;
}

// JG: the columns of J (the accumulated rotations) live in global memory (Jglobal, l columns of ldm elements, one
// such array per problem of a batch, `stride` bytes apart) instead of LDS, for orders whose two matrices do not fit
// there together (fp64 beyond 96).  Its columns travel through the cache of the CU: a round takes longer, but
// the problems of a batch still run side by side, one workgroup each.
template <typename T, typename TIn, int RPL, int G, bool JG = false, bool CORR = false>
__global__ __launch_bounds__(64 * G) void jacobi_lds_kernel(const TIn *__restrict__ M, int l, SigmaOut sig,
                                                         T *__restrict__ X, T *__restrict__ W, DevInfo *info,
                                                         int64_t stride, int rows, T *__restrict__ Jglobal) {
  extern __shared__ __attribute__((aligned(16))) double lds_raw[];
  if (blockIdx.x != 0) {              // batched launch: one problem per workgroup, `stride` bytes apart
    const int64_t off = (int64_t)blockIdx.x * stride;
    M = reinterpret_cast<const TIn *>(reinterpret_cast<const char *>(M) + off);
    X = reinterpret_cast<T *>(reinterpret_cast<char *>(X) + off);
    W = reinterpret_cast<T *>(reinterpret_cast<char *>(W) + off);
    if (JG) Jglobal = reinterpret_cast<T *>(reinterpret_cast<char *>(Jglobal) + off);
  }
  const int ldm = jacobi_ldm(l, G, (int)sizeof(T));
  T *Mc = reinterpret_cast<T *>(lds_raw);
  T *Jc = JG ? Jglobal : Mc + (size_t)l * ldm;
  T *B0 = Mc + (size_t)(JG ? 1 : 2) * l * ldm, *B1 = B0 + (CORR ? (l + 15) / 16 * 16 * corr_ld(l) : 0);      // (work of the corrections)
  T *nrm = B1 + (B1 - B0);
  int *rnk = reinterpret_cast<int *>(nrm + l);
  __shared__ int rotations;
  __shared__ unsigned turned_sum;
  __shared__ T wave_sum[16];
  __shared__ __attribute__((aligned(16))) JacLevel lev[kJacLevels][kJacGroups];
  static_assert(!CORR || (!JG && CorrCfg<T, RPL>::kFits), "no room for the matrices of the corrections");
  __shared__ double corr_norms[CORR ? 16 * RPL : 1];
  __shared__ f32x4 corr_sums[CORR ? kCorrWaves : 1];

  const int tid = threadIdx.x, nt = blockDim.x;
  // pair order: every column finds, level by level, the set it belongs to; the columns of
  // a front half claim lane group (start of the set) / 2 + (position in the half)
  for (int e = tid; e < kJacLevels * kJacGroups; e += nt) (&lev[0][0])[e].stat = 255;
  __syncthreads();
  if (tid < l) {
    int start = 0, size = l;
    for (int d = 0; d < kJacLevels && size > 1; ++d) {
      const int h = size >> 1;
      if (tid < start + h) {
        JacLevel e;
        e.stat = (unsigned char)tid; e.bstart = (unsigned char)(start + h); e.bsize = (unsigned char)(size - h);
        e.idx = (unsigned char)(tid - start);
        lev[d][(start >> 1) + (tid - start)] = e;
        size = h;
      } else {
        start += h;
        size -= h;
      }
    }
  }
  T fro2 = 0;
  {
    // M is row-major in global memory and column-major in LDS: consecutive threads take consecutive elements
    // of a row (one cache line per 16 or 8 of them); the padding rows of the columns are cleared apart
    const int pad = ldm - l;
    for (int idx = tid; idx < l * pad; idx += nt) {
      const int c = idx / pad, r = l + (idx - c * pad);
      Mc[c * ldm + r] = (T)0;
      Jc[c * ldm + r] = (T)0;
    }
    // (what lies between the rows of the corrections' matrices is read as columns of J beyond the last one, against zeros: it has to be finite)
    if (CORR) {
      for (T *w = B0 + tid; w < nrm; w += nt) *w = (T)0;
      if (tid < kCorrWaves) corr_sums[tid] = f32x4{0.f, 0.f, 0.f, 0.f};       // (as many are added up, with fewer wavefronts as well)
    }
    for (int idx = tid; idx < l * l; idx += nt) {
      const int r = idx / l, c = idx - r * l;
      const T v = (T)M[idx];
      if (rows) Mc[r * ldm + c] = v;                      // the rows of M are what is rotated: M^T is decomposed
      else Mc[c * ldm + r] = v;
      Jc[c * ldm + r] = (r == c) ? (T)1 : (T)0;
      fro2 += v * v;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) fro2 += __shfl_xor(fro2, off, 64);
  if ((tid & 63) == 0) wave_sum[tid >> 6] = fro2;
  if (tid == 0) { rotations = 0; turned_sum = 0; }
  __syncthreads();
  fro2 = 0;
  for (int w = 0; w < (nt >> 6); ++w) fro2 += wave_sum[w];
  // Scale M by a power of two to ||M||_F ~ 1 (exact; undone when sigma is written): products of squared
  // column norms then stay inside the range of the type whatever the scale of the input.
  T unscale = (T)1;
  if (fro2 > (T)0 && fro2 < (T)3e38) {
    int ex;
    (void)frexp((double)fro2, &ex);                       // fro2 = f 2^ex, 1/2 <= f < 1
    const T sc = (T)ldexp(1.0, -(ex / 2));
    unscale = (T)ldexp(1.0, ex / 2);
    for (int idx = tid; idx < l * ldm; idx += nt) Mc[idx] *= sc;
    fro2 *= sc * sc;
    __syncthreads();
  }
  const T floor2 = Eps<T>::value * Eps<T>::value * fro2;

  const int group = tid / G, lg = tid % G;       // G lanes per column pair
  const T tol = Eps<T>::value * sqrt((T)l);
  int sweeps = 0, applied = 0;                   // (applied: corrections)
  bool converged = (l < 2);
  float rho_prev = -1.f;
  bool corrections = CORR;
  float turned_limit = corr_turned(l);           // (of the angles' Frobenius norm in a sweep, for a look at corrections)
  constexpr int NV = RPL / (8 / (int)sizeof(T));
  while (!converged && sweeps < kJacobiMaxSweeps) {
    ++sweeps;
    float rho = 0.f, turned = 0.f;
    int d = 0;
    for (int ms = l; ms > 1; ms = (ms + 1) >> 1, ++d) {      // ms: largest set of this level
      JacLevel e;
      e.stat = 255; e.bstart = 0; e.bsize = 0; e.idx = 0;
      if (group < kJacGroups) e = lev[d][group];
      const bool act = e.stat != 255;
      jac_unit<T> x[NV], u[NV];
      if (act) {
        load_column<T, RPL, G>(Mc + e.stat * ldm, lg, x);
        load_column<T, RPL, G>(Jc + e.stat * ldm, lg, u);
      }
      const int nr = ms - (ms >> 1);
      for (int r = 0; r < nr; ++r) {
        if (act && r < e.bsize) {
          int j = e.idx + r;
          if (j >= e.bsize) j -= e.bsize;
          rho = fmaxf(rho, rotate_moving<T, RPL, G>(x, u, Mc, Jc, ldm, e.bstart + j, lg, tol, floor2, turned));
        }
        __syncthreads();
      }
      if (act) {
        store_column<T, RPL, G>(Mc + e.stat * ldm, lg, x);
        store_column<T, RPL, G>(Jc + e.stat * ldm, lg, u);
      }
      __syncthreads();
    }
    if (rho > 0.f) {
      atomicMax(&rotations, __float_as_int(rho));      // positive floats order like their bit patterns
      // (whole numbers: their sum does not depend on the order)
      if (CORR && lg == 0) atomicAdd(&turned_sum, (unsigned)(turned * kCorrTurnedScale));
    }
    __syncthreads();
    converged = jacobi_done(__int_as_float(rotations), rho_prev, (float)tol);
    rho_prev = __int_as_float(rotations);
    const float turned_all = CORR ? sqrtf(2.f / kCorrTurnedScale * (float)turned_sum) : 0.f;
    __syncthreads();
    if (tid == 0) { rotations = 0; turned_sum = 0; }
    __syncthreads();
    if constexpr (CORR) {
      if (!converged && corrections && turned_all <= turned_limit) {
        converged = lds_corrections<T, RPL>(Mc, Jc, ldm, B0, B1, l, tol, floor2, corr_norms, corr_sums, applied);
        // Corrections that did not get there have met a cluster, whose angles stay large however small the inner products: the rest is left to
        // sweeps, about whose rate the ones before say nothing.
        if (applied > 0) { rho_prev = -1.f; corrections = false; }
        else turned_limit = 0.5f * turned_all;
      }
    }
  }

  // Norms of the columns of M, sixteen lanes each.  Those of J are not quite one: the rounding errors of c and s err to one side where the
  // angles are large and, less, to the other where they are small (fp64, l = 61: J^T J - I -31 eps on the diagonal behind five sweeps, -5 behind
  // eight), and M has the same factors.  They are taken out of both (largest error of a value, factor of a
  // Gaussian matrix, fp64 l = 61 6.8 -> 3.6 eps, over six decades 40 -> 4.0; fp32 l = 80 7.8 -> 2.1).
  static_assert(sizeof(lev) >= 128 * sizeof(T), "one factor for each column");
  T *unit = reinterpret_cast<T *>(&lev[0][0]);        // (the pair order is no longer needed)
  for (int j = tid >> 4; j < l; j += nt >> 4) {
    double sm = 0.0, sj = 0.0;
    for (int r = tid & 15; r < l; r += 16) {
      const double x = (double)Mc[j * ldm + r], u = (double)Jc[j * ldm + r];
      sm += x * x;
      sj += u * u;
    }
    sm = group_sum<16>(sm);
    sj = group_sum<16>(sj);
    if ((tid & 15) == 0) {
      unit[j] = (T)(1.5 - 0.5 * sj);
      nrm[j] = (T)(sqrt(sm) * (1.5 - 0.5 * sj));
    }
  }
  __syncthreads();
  for (int j = tid; j < l; j += nt) {
    const T mine = nrm[j];
    int rank = 0;
    for (int i = 0; i < l; ++i) {
      const T o = nrm[i];
      rank += (o > mine || (o == mine && i < j)) ? 1 : 0;
    }
    rnk[j] = rank;
    if (rank < sig.n) reinterpret_cast<T *>(reinterpret_cast<char *>(sig.p) + (int64_t)blockIdx.x * sig.stride)[rank] = mine * unscale;
  }
  __syncthreads();
  for (int idx = tid; idx < l * l; idx += nt) {
    const int r = idx / l, c = idx - r * l;
    const int dst = r * l + rnk[c];
    const T s = nrm[c];
    X[dst] = (s * s > floor2) ? Mc[c * ldm + r] * unit[c] / s : (T)0;
    W[dst] = Jc[c * ldm + r] * unit[c];
  }
  if (tid == 0 && info != nullptr) {
    atomicMax(&info->jacobi_sweeps, sweeps + applied);
    if (!converged) atomicMax(&info->status, (int)RSVD_ERR_NO_CONVERGENCE);
  }
}

// ---------------------------------------------------------------- orders beyond one workgroup's LDS
//
// Block one-sided Jacobi.  M^T and J^T live in global memory (column c of M is
// row c of Mt, contiguous).  The columns are cut into blocks of b; an outer
// sweep is a round-robin tournament over the blocks, one workgroup per block pair.
// Orders whose panel of 2b columns fits in LDS take one launch for all sweeps
// (jb_flow_kernel, rotations from the Gram matrix of the panel).  Longer columns
// take one launch per round (jb_panel_kernel): the workgroup rotates its columns pair
// by pair, accumulates the rotations in a small 2b x 2b matrix T, writes the columns
// back and leaves T for the matching columns of J.
// counters[s] collects the largest relative inner product that outer sweep s
// rotated away; sweeps that the ones before make unnecessary (jacobi_done) are left
// out by the kernels themselves, which keeps the whole sequence free of host
// synchronisation.

// Sum over the 32 lanes of a pair group: the 16-lane row by DPP (neighbours, pairs,
// half-row mirror, row mirror), then one exchange with the partner row.
template <typename T> __device__ __forceinline__ T group32_sum(T v) {
#pragma clang fp contract(off)
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v += dpp_mov<0x141>(v);
  v += dpp_mov<0x140>(v);
  v += __shfl_xor(v, 16, 32);
  return v;
}

// Panel version of rotate_pair: columns of length up to 32 * NV units held in LDS
// (stride ldp, zero padded), 32 lanes per pair, the accumulated rotation T
// (rows_t x rows_t, stride ldt) instead of J.
template <typename T, int NV>
__device__ __forceinline__ float rotate_pair_panel(T *Pc, T *Tc, int ldp, int ldt, int rows_t, int p, int q, int lg,
                                                  T tol, T floor2) {
  constexpr int V = 8 / sizeof(T);
  typedef T unit __attribute__((ext_vector_type(V)));
  unit *mp = reinterpret_cast<unit *>(Pc + p * ldp) + lg;
  unit *mq = reinterpret_cast<unit *>(Pc + q * ldp) + lg;
  unit x[NV], y[NV];
#pragma unroll
  for (int r = 0; r < NV; ++r) { x[r] = mp[32 * r]; y[r] = mq[32 * r]; }
  T alpha = 0, beta = 0, gamma = 0;
#pragma unroll
  for (int r = 0; r < NV; ++r)
#pragma unroll
    for (int e = 0; e < V; ++e) {
      alpha += x[r][e] * x[r][e];
      beta += y[r][e] * y[r][e];
      gamma += x[r][e] * y[r][e];
    }
  alpha = group32_sum(alpha);
  beta = group32_sum(beta);
  gamma = group32_sum(gamma);
  if (alpha <= floor2 || beta <= floor2) return 0.f;
  const T rel = fabs(gamma) * fast_rsq(alpha * beta);        // |x.y| / (|x| |y|); the matrix was scaled to unit size
  if (!(rel > tol)) return 0.f;
  const float ratio = (float)rel;
  T c, s;
  rotation_params(alpha, beta, gamma, c, s);
#pragma unroll
  for (int r = 0; r < NV; ++r) {
    mp[32 * r] = c * x[r] - s * y[r];
    mq[32 * r] = s * x[r] + c * y[r];
  }
  T *tp = Tc + p * ldt, *tq = Tc + q * ldt;
  for (int i = lg; i < rows_t; i += 32) {
    const T a = tp[i], bq = tq[i];
    tp[i] = c * a - s * bq;
    tq[i] = s * a + c * bq;
  }
  return ratio;
}

// Cross-phase version: the column of the first block (x, NV units per lane) and its
// column of T (tx: entries lg and lg + 32) stay in registers for all rounds of the launch;
// only the column of the second block (qp: its place in LDS) and its column qt of T go through LDS.
template <typename T, int NV>
__device__ __forceinline__ float rotate_moving_panel(jac_unit<T> (&x)[NV], T (&tx)[2], T *Pc, T *Tc, int ldp, int ldt,
                                                    int rows_t, int qp, int qt, int lg, T tol, T floor2) {
  constexpr int V = 8 / sizeof(T);
  jac_unit<T> *mq = reinterpret_cast<jac_unit<T> *>(Pc + qp * ldp) + lg;
  jac_unit<T> y[NV];
#pragma unroll
  for (int r = 0; r < NV; ++r) y[r] = mq[32 * r];
  T alpha = 0, beta = 0, gamma = 0;
#pragma unroll
  for (int r = 0; r < NV; ++r)
#pragma unroll
    for (int e = 0; e < V; ++e) {
      alpha += x[r][e] * x[r][e];
      beta += y[r][e] * y[r][e];
      gamma += x[r][e] * y[r][e];
    }
  alpha = group32_sum(alpha);
  beta = group32_sum(beta);
  gamma = group32_sum(gamma);
  if (alpha <= floor2 || beta <= floor2) return 0.f;
  const T rel = fabs(gamma) * fast_rsq(alpha * beta);        // |x.y| / (|x| |y|); the matrix was scaled to unit size
  if (!(rel > tol)) return 0.f;
  const float ratio = (float)rel;
  T c, s;
  rotation_params(alpha, beta, gamma, c, s);
#pragma unroll
  for (int r = 0; r < NV; ++r) {
    const jac_unit<T> xo = x[r];
    x[r] = c * xo - s * y[r];
    mq[32 * r] = s * xo + c * y[r];
  }
  T *tq = Tc + qt * ldt;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int i = lg + 32 * j;
    if (i < rows_t) {
      const T a = tx[j], bq = tq[i];
      tx[j] = c * a - s * bq;
      tq[i] = s * a + c * bq;
    }
  }
  return ratio;
}

// scratch header shared by the block-Jacobi kernels
constexpr int kJbFroParts = 64;
struct JbHeader {
  double fro2;            // ||M||_F^2 of the scaled matrix
  double unscale;         // the singular values of M are those of the scaled matrix times this
  int counters[64];       // jb_panel_kernel, per outer sweep: bit pattern of the largest relative inner product rotated away
  double partial[kJbFroParts];   // sums of squares, one per workgroup of jb_fro_kernel
};

// One run of sweeps of jb_flow_kernel.
constexpr int kRunSweeps = 64;
static_assert(kJacobiMaxSweeps <= kRunSweeps, "a record for every sweep");
struct JbRun {
  unsigned long long sumsq[kRunSweeps];      // per sweep: sum of s^2 over its rotations (c, s), times kJbSumScale
  int counters[kRunSweeps];                  // per sweep: bit pattern of the largest relative inner product rotated away
  int finished[kRunSweeps];                  // per sweep: block pairs whose columns of M are done
  int ticket;                        // next task
  int stop;                          // 1: converged, 2: what is left is for the corrections of the whole matrix
  int used;                          // sweeps done when it stopped
  int pad;
};
constexpr int kPolishPhases = 13;
// The corrections of the whole matrix behind the first run, and the run behind those.
struct JbSync {
  JbRun run[2];
  unsigned long long x2[kPolishSteps];      // per correction: sum of the squared angles of all pairs times kPolishScale
  unsigned long long x2_open[kPolishSteps]; // and of the pairs above the threshold of a rotation
  int rho[kPolishSteps];                    // and the largest relative inner product it found
  int done[kPolishSteps * kPolishPhases];   // tiles finished, phase by phase
  int updates, converged;                   // how the corrections ended
  int ticket, pad;                          // next tile
  double fro2, unscale;                     // as in JbHeader
};
static_assert(sizeof(JbSync) % 8 == 0 && sizeof(JbSync) <= 4096, "lies at the start of an l x l slot");
constexpr float kJbSumScale = 65536.f;

// ||M||_F^2 in kJbFroParts partial sums (fixed assignment of elements and fixed order: reproducible).
__global__ __launch_bounds__(256) void jb_fro_kernel(const double *__restrict__ M, int l, JbHeader *hdr) {
  __shared__ double wave_sum[4];
  const int tid = threadIdx.x;
  double s2 = 0;
  for (int64_t idx = (int64_t)blockIdx.x * 256 + tid; idx < (int64_t)l * l; idx += (int64_t)kJbFroParts * 256) {
    const double v = M[idx];
    s2 += v * v;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s2 += __shfl_xor(s2, off, 64);
  if ((tid & 63) == 0) wave_sum[tid >> 6] = s2;
  __syncthreads();
  if (tid == 0) hdr->partial[blockIdx.x] = (wave_sum[0] + wave_sum[1]) + (wave_sum[2] + wave_sum[3]);
}

// Mt = (sc M)^T in the working type, Jt = I, with sc the power of two that brings ||M||_F to ~1 (exact, undone
// when the singular values are written): products of squared column norms then stay inside the range of
// the type whatever the scale of the input.  Grid of workgroups, each taking a slab of elements.
template <typename T>
__global__ __launch_bounds__(256) void jb_init_kernel(const double *__restrict__ M, int l, T *__restrict__ Mt,
                                                      T *__restrict__ Jt, JbHeader *hdr, int rows,
                                                      int *__restrict__ ver, int nver, JbSync *sync, int *__restrict__ ver2) {
  double fro2 = 0;
  for (int i = 0; i < kJbFroParts; ++i) fro2 += hdr->partial[i];
  double sc = 1.0, unscale = 1.0;
  if (fro2 > 0.0 && fro2 <= 1.79e308) {
    int ex;
    (void)frexp(fro2, &ex);
    sc = ldexp(1.0, -(ex / 2));
    unscale = ldexp(1.0, ex / 2);
  }
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < (int64_t)l * l;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int r = (int)(idx / l), c = (int)(idx - (int64_t)r * l);
    Mt[rows ? idx : (int64_t)c * l + r] = (T)(M[idx] * sc);      // rows: M^T is decomposed, its columns are M's rows
    Jt[idx] = (r == c) ? (T)1 : (T)0;
  }
  if (blockIdx.x == 0) {
    if (threadIdx.x < 64) hdr->counters[threadIdx.x] = 0;
    for (int i = threadIdx.x; i < nver; i += blockDim.x) ver[i] = 0;
    if (sync != nullptr) {
      int *p = reinterpret_cast<int *>(sync);
      for (int i = threadIdx.x; i < (int)(offsetof(JbSync, fro2) / sizeof(int)); i += blockDim.x) p[i] = 0;
      for (int i = threadIdx.x; i < nver; i += blockDim.x) ver2[i] = 0;
    }
    if (threadIdx.x == 0) {
      hdr->fro2 = fro2 * sc * sc;
      hdr->unscale = unscale;
      if (sync != nullptr) {
        sync->fro2 = fro2 * sc * sc;
        sync->unscale = unscale;
      }
    }
  }
}

// Padded column length (elements) of the panel layout: 32 lanes x NV units.
template <typename T, int NV> __host__ __device__ constexpr int jb_ldp() { return 32 * NV * (8 / (int)sizeof(T)) + 2; }

// phase 0 ("diagonal"): workgroup g rotates the pairs inside column block g
//   (cols - 1 rounds of the circle tournament).
// phase 1 ("cross"): workgroup g takes the block pair g of tournament round `round`
//   and rotates only pairs with one column in each block: b rounds, pair i of
//   round r is (i, (i + r) mod b) - every column of one block meets every column of
//   the other exactly once.
// One outer sweep = one diagonal launch + (nblk - 1) cross launches = l - 1 rounds
// in all, the same count as the plain tournament.
//
// The rotations never read J, and a launch keeps only nblk / 2 of the chip's workgroups busy.
// So a rotating workgroup only leaves its accumulated T (and a flag that it rotated at all) in a
// two-slot ring in global memory, and the NEXT launch carries, behind its own rot_wgs rotating
// workgroups, one workgroup per (block pair of the launch before, chunk of kJbRowChunk rows) that
// applies that T to the matching columns of J on the matrix cores while the rotations of the
// current round run.  A last launch with rot_wgs = 0 applies what the final round left.

// Block pair (and column counts) of workgroup g of a launch.
struct JbPair { int bi, bj, cols_i, cols_j; bool valid; };
__device__ __forceinline__ JbPair jb_pair(int phase, int round, int g, int l, int b, int nblk) {
  JbPair p;
  p.valid = true;
  if (phase == 0) {
    p.bi = p.bj = g;
    p.cols_i = (l - p.bi * b < b) ? (l - p.bi * b) : b;
    p.cols_j = 0;
  } else {
    const int nblk2 = nblk + (nblk & 1);
    int ba, bb;
    tournament_pair(nblk2, round, g, ba, bb);
    p.valid = ba < nblk && bb < nblk;                          // else a bye
    p.bi = ba < bb ? ba : bb;
    p.bj = ba < bb ? bb : ba;
    p.cols_i = (l - p.bi * b < b) ? (l - p.bi * b) : b;
    p.cols_j = p.valid ? ((l - p.bj * b < b) ? (l - p.bj * b) : b) : 0;
  }
  return p;
}

constexpr int kJbRowChunk = 64;      // one row per lane of a wavefront when the chunk is staged (jb_apply_t)

// J[rows of chunk, panel] <- J[rows of chunk, panel] T for block pair `pr`: the old entries staged
// through LDS, a (64 x 2b) by (2b x 2b) product in 16 x 16 blocks.
template <typename T>
__device__ __forceinline__ void jb_apply_t(T *__restrict__ Jt, const T *__restrict__ Tg, int l, int b, const JbPair &pr,
                                           int chunk, T *lds) {
  static_assert(kJbRowChunk == 64, "the staging loop below moves one row per lane of a wavefront");
  constexpr int LDJ = kJbRowChunk + 8;
  const int ldt = 2 * b + 2;
  T *Pj = lds;                       // [2b][LDJ]: Pj[k][i] = J[i0 + i][panel column k]
  T *Tl = lds + (size_t)(2 * b) * LDJ;      // [2b][ldt]: Tl[col][k] = T[k][col]
  const int tid = threadIdx.x, nt = blockDim.x;
  const int lane64 = tid & 63, wave = tid >> 6, nwave = nt >> 6;
  const int ncols = pr.cols_i + pr.cols_j;
  const int i0 = chunk * kJbRowChunk;
  auto gcol = [&](int c) { return c < pr.cols_i ? pr.bi * b + c : pr.bj * b + (c - pr.cols_i); };
  for (int c = wave; c < 2 * b; c += nwave) {
    const int i = i0 + lane64;
    Pj[c * LDJ + lane64] = (c < ncols && i < l) ? Jt[(int64_t)gcol(c) * l + i] : (T)0;
  }
  for (int idx = tid; idx < 4 * b * b; idx += nt) {
    const int c = idx / (2 * b), k = idx - c * (2 * b);
    Tl[c * ldt + k] = Tg[idx];
  }
  __syncthreads();
  typedef typename Mfma<T>::vec acc_t;
  const int r16 = lane64 & 15, kq = lane64 >> 4;
  const int col_blocks = (2 * b) / 16;
  for (int blk = wave; blk < (kJbRowChunk / 16) * col_blocks; blk += nwave) {
    const int rb = blk / col_blocks, cb = blk - rb * col_blocks;
    acc_t acc = (acc_t)(T)0;
    const T *ap = Pj + kq * LDJ + rb * 16 + r16;                  // Jold[row][k]
    const T *bp = Tl + (cb * 16 + r16) * ldt + kq;                // T[k][col]
#pragma unroll 4
    for (int k0 = 0; k0 < 2 * b; k0 += 4) acc = Mfma<T>::run(ap[k0 * LDJ], bp[k0], acc);
    const int cn = cb * 16 + r16;
    if (cn < ncols) {
      T *dst = Jt + (int64_t)gcol(cn) * l;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = i0 + rb * 16 + Mfma<T>::row(lane64, v);
        if (r < l) dst[r] = acc[v];
      }
    }
  }
}

// J role of a launch: workgroup j behind the rot_wgs rotating ones applies the T that block pair g of the launch
// before (phase, round, sweep = prev_*) left in the other slot of the ring to one chunk of rows of J.
template <typename T>
__device__ __forceinline__ void jb_j_role(T *__restrict__ Jt, int l, int b, int nblk, int rot_wgs, int prev_phase,
                                          int prev_round, int prev_sweep, const T *__restrict__ Tring,
                                          const int *__restrict__ chg, int slot, const JbHeader *hdr, float tol,
                                          T *lds) {
  const int chunks = (l + kJbRowChunk - 1) / kJbRowChunk;
  const int j = (int)blockIdx.x - rot_wgs;
  const int g = j / chunks;
  if (jacobi_done_before(hdr->counters, prev_sweep, tol)) return;                  // that launch did nothing
  const JbPair pr = jb_pair(prev_phase, prev_round, g, l, b, nblk);
  const int pslot = slot ^ 1;
  if (!pr.valid || chg[pslot * nblk + g] == 0) return;
  jb_apply_t<T>(Jt, Tring + ((size_t)pslot * nblk + g) * (size_t)(4 * b * b), l, b, pr, j - g * chunks, lds);
}

template <typename T, int NV>
__global__ __launch_bounds__(1024) void jb_panel_kernel(T *__restrict__ Mt, T *__restrict__ Jt, int l, int b,
                                                        int nblk, int phase, int round, int sweep, int rot_wgs,
                                                        int prev_phase, int prev_round, int prev_sweep,
                                                        T *__restrict__ Tring, int *__restrict__ chg, int slot,
                                                        JbHeader *hdr) {
  const T tol = Eps<T>::value * sqrt((T)l);
  extern __shared__ __attribute__((aligned(16))) double lds_raw[];
  if ((int)blockIdx.x >= rot_wgs) {
    jb_j_role<T>(Jt, l, b, nblk, rot_wgs, prev_phase, prev_round, prev_sweep, Tring, chg, slot, hdr, (float)tol,
                 reinterpret_cast<T *>(lds_raw));
    return;
  }
  if (jacobi_done_before(hdr->counters, sweep, (float)tol)) return;        // the sweeps before finished the job
  const JbPair pr = jb_pair(phase, round, (int)blockIdx.x, l, b, nblk);
  if (!pr.valid) return;                                       // bye
  const int bi = pr.bi, bj = pr.bj, cols_i = pr.cols_i, cols_j = pr.cols_j;
  const int ncols = cols_i + cols_j;

  constexpr int ldp = jb_ldp<T, NV>();
  const int ldt = (2 * b) + 2;
  // LDS holds ONE block of columns: the block itself in the diagonal phase, the second ("moving")
  // block in the cross phase, whose first block lives in registers from global memory to global
  // memory.
  T *Pc = reinterpret_cast<T *>(lds_raw);
  T *Tc = Pc + (size_t)b * ldp;
  __shared__ int rotations;
  const int lds_blk = (phase == 0) ? bi : bj;
  const int lds_cols = (phase == 0) ? cols_i : cols_j;

  const int tid = threadIdx.x, nt = blockDim.x;
  // panel in: a wavefront takes whole columns, two at a time, and issues every load of both
  // before the first LDS store (the loads are the latency to hide)
  constexpr int LPW = (ldp + 63) / 64;      // elements per lane per column
  const int lane64 = tid & 63, wave = tid >> 6, nwave = nt >> 6;
  auto panel_in = [&](const T *__restrict__ G) {
    for (int c0 = wave; c0 < b; c0 += 2 * nwave) {
      T v[2][LPW];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int c = c0 + u * nwave;
        const T *src = G + (int64_t)(lds_blk * b + (c < lds_cols ? c : 0)) * l;
#pragma unroll
        for (int j = 0; j < LPW; ++j) {
          const int r = lane64 + 64 * j;
          v[u][j] = (c < lds_cols && r < l) ? src[r] : (T)0;
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int c = c0 + u * nwave;
        if (c < b) {
#pragma unroll
          for (int j = 0; j < LPW; ++j) {
            const int r = lane64 + 64 * j;
            if (r < ldp) Pc[c * ldp + r] = v[u][j];
          }
        }
      }
    }
  };
  auto panel_out = [&](T *__restrict__ G) {
    for (int c = wave; c < lds_cols; c += nwave) {
      T *dst = G + (int64_t)(lds_blk * b + c) * l;
#pragma unroll
      for (int j = 0; j < LPW; ++j) {
        const int r = lane64 + 64 * j;
        if (r < l) dst[r] = Pc[c * ldp + r];
      }
    }
  };
  panel_in(Mt);
  for (int idx = tid; idx < 2 * b * ldt; idx += nt) {
    const int c = idx / ldt, r = idx - c * ldt;
    Tc[idx] = (r == c && c < ncols) ? (T)1 : (T)0;
  }
  if (tid == 0) rotations = 0;

  const T floor2 = (T)(Eps<T>::value * Eps<T>::value * hdr->fro2);
  const int group = tid >> 5, lg = tid & 31;                   // 32 groups of 32 lanes, b <= 32
  constexpr int V = 8 / (int)sizeof(T);
  float rho = 0.f;
  // cross phase: lane group g keeps column g of the first block (and its column of T) for all b rounds
  const bool act = phase != 0 && group < cols_i;
  jac_unit<T> x[NV];
  T tx[2] = {(T)0, (T)0};
  if (act) {
    const T *src = Mt + (int64_t)(bi * b + group) * l;
#pragma unroll
    for (int r = 0; r < NV; ++r)
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const int row = (lg + 32 * r) * V + e;
        x[r][e] = row < l ? src[row] : (T)0;
      }
#pragma unroll
    for (int j = 0; j < 2; ++j) tx[j] = (lg + 32 * j == group) ? (T)1 : (T)0;     // column `group` of the identity
  }
  __syncthreads();

  if (phase == 0) {
    const int n2 = ncols + (ncols & 1);
    for (int r = 0; r < n2 - 1; ++r) {
      if (group < n2 / 2) {
        int a, c2;
        tournament_pair(n2, r, group, a, c2);
        if (a < ncols && c2 < ncols) {
          const int p = a < c2 ? a : c2, q = a < c2 ? c2 : a;
          rho = fmaxf(rho, rotate_pair_panel<T, NV>(Pc, Tc, ldp, ldt, ncols, p, q, lg, tol, floor2));
        }
      }
      __syncthreads();
    }
  } else {
    for (int r = 0; r < b; ++r) {
      int qi = group + r;
      if (qi >= b) qi -= b;
      if (act && qi < cols_j)
        rho = fmaxf(rho, rotate_moving_panel<T, NV>(x, tx, Pc, Tc, ldp, ldt, ncols, qi, cols_i + qi, lg, tol, floor2));
      __syncthreads();
    }
    if (act) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
        if (lg + 32 * j < ncols) Tc[group * ldt + lg + 32 * j] = tx[j];
    }
    __syncthreads();
  }
  if (rho > 0.f) atomicMax(&rotations, __float_as_int(rho));
  __syncthreads();
  const int rho_bits = rotations;
  if (rho_bits == 0) {                                        // nothing changed: leave M alone, no T to apply
    if (tid == 0) chg[slot * nblk + blockIdx.x] = 0;
    return;
  }
  panel_out(Mt);
  if (act) {
    T *dst = Mt + (int64_t)(bi * b + group) * l;
#pragma unroll
    for (int r = 0; r < NV; ++r)
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const int row = (lg + 32 * r) * V + e;
        if (row < l) dst[row] = x[r][e];
      }
  }
  T *Tg = Tring + ((size_t)slot * nblk + blockIdx.x) * (size_t)(4 * b * b);
  for (int idx = tid; idx < 4 * b * b; idx += nt) {
    const int c = idx / (2 * b), k = idx - c * (2 * b);
    Tg[idx] = Tc[c * ldt + k];
  }
  if (tid == 0) {
    chg[slot * nblk + blockIdx.x] = 1;
    atomicMax(&hdr->counters[sweep], rho_bits);
  }
}

// ---- all sweeps in one launch, rotations from the Gram matrix of a block pair ----
//
// Rotating 2b columns of length l column by column (jb_panel_kernel) costs ~1 us of plain vector instructions a round
// whatever l is.  The rotations only need inner products, and those follow from the 2b x 2b Gram matrix G of the panel:
// G is formed once on the matrix cores, the rounds rotate G on both sides (G <- J^T G J, a 2 x 2 block per thread) and
// accumulate T <- T J, and the panel is multiplied by T once, again on the matrix cores.  Rotation formulas, thresholds
// and the stopping rule are those of the column-by-column kernel; the first round sees exact inner products, later
// rounds the tracked ones (their error is of second order in the rotation angles and is wiped out by the next visit,
// which forms G afresh).  T is accumulated in fp64 and rounded once: an error of its large elements is common to a whole
// column, where the errors of rotated columns average out, and those of (c, s) and of the updates in fp32 point the same way for
// thousands of rotations (singular values off by 5.4, 11.5 and 21.6 eps at l = 129, 300, 576, rms, geometric mean over five kinds of spectrum; now 1.2,
// 1.4 and 1.7; up to 1 % more time).
//
// A sweep is a tournament over the column blocks: nblk2 - 1 steps of nblk2 / 2 block pairs.  A pair's task rotates the
// b x b pairs of columns across its two blocks (b rounds: pair i of round r is (i, b + (i + r) mod b)), in the first step
// of a sweep also the pairs inside either block before them (b - 1 rounds of the circle method, both blocks side by
// side); then it applies T to the matching columns of J.
//
// Tasks are numbered in the order sweep, step, pair and handed out by a counter; a task waits until its blocks have
// been through the step before (ver: M, ver + nblk: J), the tasks of the first step of a sweep until the sweep before is
// complete, whose record says whether there is anything left to do.  Every wait is for tasks with lower numbers, whose
// workgroups are running already, so the lowest unfinished task never waits for anything unfinished: no number of
// resident workgroups is assumed, and no other kernel on the chip can stop the progress.  M and J are read and
// written with device-wide scope (the L2 caches of the XCDs do not see each other's lines).  J is off the critical
// path: the columns of M are published before it is touched, and with two workgroups per block pair the next step
// runs meanwhile.
//
// What bounds a step is its chain: panel in 2.1 us, G 3.0, 16 rounds of ~0.4 (fp64; 0.3 in fp32), panel out 1.9, the
// stores' arrival 1.3, the wait for them elsewhere ~1 (fp64, l = 288).  Against one launch per step with the rotations of
// J a step behind (the launches of sweeps that are not needed come to a quarter of the time): whole decomposition
// of the triangular factor of a Gaussian matrix of l + 37 rows, 9 to 10 sweeps (8 at l = 210): 1526 -> 1018 us (fp64, l = 128), 4115 -> 2844
// (fp64, 288), 2147 -> 1446 (fp32, 210), 7834 -> 5164 (fp32, 576).
constexpr int kJgB = 16;                    // block width this kernel is written for
constexpr int kJgN = 2 * kJgB;              // columns of a panel
constexpr int kJgLd = kJgN + 1;             // row stride of G and T in LDS
constexpr int kJgMat = kJgN * kJgLd;        // elements of one such matrix
constexpr int kJgPart = 3 * 256;            // elements of one partial sum of G (three 16 x 16 blocks)
template <bool V> struct JbKind { static constexpr bool value = V; };

// Column stride of the panel in LDS: l padded to whole 16-row blocks, plus what spreads sixteen 16-byte pieces of 16
// columns over the banks.
template <typename T> __host__ __device__ constexpr int jg_ldp(int l) {
  return (l + 15) / 16 * 16 + 16 / (int)sizeof(T);
}
template <typename T> __host__ __device__ constexpr size_t jg_lds_bytes(int l) {
  return ((size_t)kJgN * jg_ldp<T>(l) + 5 * (size_t)kJgMat) * sizeof(T);
}

// Longest columns (a wavefront stages a column through this many / 64 registers); LDS ends at about the same order.
template <typename T> __host__ __device__ constexpr int jg_max_order() { return sizeof(T) == 4 ? 1088 : 512; }
constexpr size_t kJgLds = 160 * 1024 - 1024;      // dynamic LDS of the kernel, beside the little it has by itself
static_assert(jg_lds_bytes<float>(1088) <= kJgLds && jg_lds_bytes<float>(1089) > kJgLds, "largest fp32 order of the flow kernel");
static_assert(jg_lds_bytes<double>(464) <= kJgLds && jg_lds_bytes<double>(465) > kJgLds, "largest fp64 order of the flow kernel");

// Pair i of a round is always the columns in slots p and q of G and T; behind the round the contents of these slots move to
// slots mp and mq, so that the next round finds its pairs in the same places: no address depends on the round.  INTRA,
// pairs inside the blocks: circle method over the 16 slots of a block (slot 15 stays, the others move up by one), pairs 0-7 in
// the first block and 8-15 in the second.  Else pairs across the blocks: the second block moves down by one.  After the
// b - 1 and the b rounds every column is back in its own slot.
template <bool INTRA> __device__ __forceinline__ void jg_pair(int i, int &p, int &q, int &mp, int &mq) {
  if (INTRA) {
    const int h = i & 7, base = (i >> 3) * kJgB;
    p = base + h;
    q = base + kJgB - 1 - h;
    mp = p + 1;
    mq = h == 0 ? q : (h == 1 ? base : q + 1);
  } else {
    p = mp = i;
    q = kJgB + i;
    mq = kJgB + ((i - 1) & (kJgB - 1));
  }
}

// The columns that pair i of round r rotates.
template <bool INTRA> __device__ __forceinline__ void jg_columns(int i, int r, int &p, int &q) {
  if (INTRA) {
    const int h = i & 7, base = (i >> 3) * kJgB, n = kJgB - 1;
    const int a = h - r, b = n - h - r;                            // (r < 15: one turn at most)
    p = base + (a < 0 ? a + n : a);
    q = base + (h == 0 ? n : (b < 0 ? b + n : b));
  } else {
    p = i;
    q = kJgB + ((i + r) & (kJgB - 1));
  }
}

// Rotation of columns p and q of the panel from the tracked Gram matrix: (c, s) = (1, 0) when the pair is left alone
// (columns that are padding have norm zero); returns the relative inner product that is rotated away (0 if none).
// Without branches: the chain of dependent instructions of a round starts here.
template <typename T>
__device__ __forceinline__ float jg_pair_params(const T *G, int p, int q, T tol, T floor2, T &c, T &s) {
  const T alpha = G[p * kJgLd + p], beta = G[q * kJgLd + q], gamma = G[p * kJgLd + q];
  T rel, cc, ss;
  bool rot = (alpha > floor2) & (beta > floor2);
  if constexpr (sizeof(T) == 4) {
    rel = fabsf(gamma) * fast_rsq(alpha * beta);
    rot = rot & (rel > tol);
    // t = 2 gamma / (|delta| + sqrt(delta^2 + 4 gamma^2)) with delta = beta - alpha, c = 1 / sqrt(1 + t^2), s = c t.
    // M is scaled to norm ~1 and columns below eps of that are not rotated: with the factor 2^32 the squares neither
    // overflow nor underflow.  (A correction of c^2 + s^2 as in fp64 leaves a bias here: singular values 5e-7 too large
    // at l = 210, 1e-8 without it.)
    const T delta = (beta - alpha) * (T)4294967296.0, g2 = gamma * (T)8589934592.0;
    const T x = delta * delta + g2 * g2;
    const T t = g2 * fast_rcp(fabsf(delta) + x * fast_rsq(x));
    cc = fast_rsq((T)1 + t * t);
    ss = cc * t;
  } else {
    // From the double angle, one division less on the chain of dependent instructions: with delta = beta - alpha and
    // u = 1 / sqrt(delta^2 + 4 gamma^2), c^2 = (1 + |delta| u) / 2 and s = gamma u / c.  M is scaled to norm ~1 and
    // columns below eps of that are not rotated, so the squares neither overflow nor underflow.  (rel only meets the
    // threshold and the rate of convergence: the hardware's estimate will do.)
    rel = fabs(gamma) * __builtin_amdgcn_rsq(alpha * beta);
    rot = rot & (rel > tol);
    const T delta = beta - alpha, ad = fabs(delta), g2 = (T)2 * gamma;
    const T u = fast_rsq(delta * delta + g2 * g2);
    const T y = (T)0.5 + (T)0.5 * ad * u;
    const T ri = fast_rsq(y);
    cc = y * ri;
    ss = gamma * u * ri;
    // The estimates err to one side: c^2 + s^2 is brought to 1 within a rounding, or every column drifts the same way over
    // the thousands of rotations it goes through (|J^T J - I| at l = 130 ... 450: 1.4e-13 with this line, 1.8e-12 without).
    const T off = (T)0.5 * fma(ss, ss, fma(cc, cc, (T)-1));
    cc -= cc * off;
    ss -= ss * off;
  }
  ss = beta < alpha ? -ss : ss;
  c = rot ? cc : (T)1;
  s = rot ? ss : (T)0;
  return rot ? (float)rel : 0.f;
}

// ---- corrections of the whole matrix at once ----
//
// The last sweeps turn columns that are nearly orthogonal by small angles, and such rotations commute up to the square of
// the angles: all of them can be taken from one Gram matrix and applied together, as the orthogonal matrix exp(X) with
// X[i][j] the angle of the pair (i, j), X antisymmetric.  What remains is of second order, as behind a sweep, but a correction is
// a handful of l x l products on all CUs where a sweep is l - 1 rounds that wait for each other.  Sweeps alone -> with corrections, whole
// decomposition: triangular factor of a Gaussian matrix of l + 37 rows, fp64 l = 110 991 -> 766 us, 288 2839 -> 2265, fp32 210 1574 -> 1251,
// 450 4062 -> 3538; nearly aligned factors with s_i = exp(-3 i / l), fp64 110 581 -> 354 us, 288 1722 -> 1035, fp32 210 740 -> 477; clusters of
// relative width 1e-5 0.87 ... 1.15 times as fast.  The columns end closer to orthogonal: G is in fp64 for either type, and a correction takes
// along the small angles below the threshold of a rotation (singular vectors of 4001 x 50021, l = 210, q = 1, twelve matrices: error against
// 64 bits 2.8e-5 -> 9.2e-6).
//   G = M^T M, X;  Y = X X, Y2 = Y Y, Y3, Y4 as far as the size of X asks for;  E = exp(X) - I;  M <- M + M E, J <- J + J E.
// exp(X) of an antisymmetric X is orthogonal: the series is cut where it is so to rounding (x: the Frobenius norm of X; the same angles are met by M and J, and E keeps the relative size of its elements, so short columns of M
// keep their relative accuracy as in a sweep).  Angles, thresholds and the floor for zero columns are those of a rotation.
// The length of the series and the halvings follow from the x of ALL angles, those below the threshold of a rotation too: with many equal
// singular values they are most of it (l = 160, 96 equal values: the pairs above the threshold 4e-5, all 9e-2), and a series cut for the others'
// sum left W off orthogonality by 2e-8 in fp64.  The limit on x and the rule that it shrinks look at the pairs above the threshold alone: inside
// a cluster the others are rounding noise and do not shrink.
// A correction that meets a larger x than it may, or one that does not shrink, does nothing and leaves the rest to sweeps, as inside a
// cluster of nearly equal singular values, where the angles stay large however small the inner products.
// Everything is decided from the counters of JbSync, which are sums of whole numbers and maxima: no order of arrival shows in the result.
constexpr float kPolishScale = 140737488355328.f;            // 2^47; a tile adds at most 128, more than any correction may

// (Large angles at tiny inner products are a cluster, which sweeps turn faster.)
__device__ __forceinline__ bool sweeps_ready(unsigned long long sumsq, float rho, int l) {
  const float x2 = (float)sumsq * (2.f / kJbSumScale);
  return x2 <= polish_start(l) * polish_start(l) && (x2 <= 4.f || rho * rho >= 2.5e-9f * x2);
}

template <typename T> struct PolishParams {
  T *b[7];                   // l x l: M (column after column), J (likewise), X, Y / next M, Y2 / next J, cosine part / E, sine part / E
  JbSync *sync;
  int l, tiles;
};

constexpr int kPoTile = 32, kPoLd = kPoTile + 1;

// The sum of the four wavefronts' tiles, in a fixed order; thread t is left with elements t, t + 256, ...
template <typename T>
__device__ __forceinline__ void polish_sum(const typename Mfma<T>::vec (&acc)[2][2], T *red, T (&out)[4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15;
  __syncthreads();                       // (red may still be read from the product before)
  T *mine = red + wave * kPoTile * kPoLd;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) mine[(16 * i + Mfma<T>::row(lane, v)) * kPoLd + 16 * j + r16] = acc[i][j][v];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int e = threadIdx.x + 256 * u, at = (e >> 5) * kPoLd + (e & 31);
    out[u] = (red[at] + red[kPoTile * kPoLd + at]) + (red[2 * kPoTile * kPoLd + at] + red[3 * kPoTile * kPoLd + at]);
  }
}

// A 32 x 32 tile of sum_k fa(k, i) fb(k, j): the four wavefronts share the k range, lane L supplies k = L / 16 of a group of four and
// i, j = L % 16 + 16 h.
template <typename T, typename FA, typename FB>
__device__ __forceinline__ void polish_tile(int l, FA fa, FB fb, T *red, T (&out)[4]) {
  typedef typename Mfma<T>::vec acc_t;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, kq = lane >> 4;
  const int groups = (l + 3) / 4, per = (groups + 3) / 4;
  const int g0 = wave * per, g1 = g0 + per < groups ? g0 + per : groups;
  acc_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = (acc_t)(T)0;
  constexpr int U = sizeof(T) == 4 ? 14 : 10;
  const int last = 4 * g1 < l ? 4 * g1 : l;
  for (int g = g0; g < g1; g += U) {
    T a[U][2], b[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = 4 * (g + u) + kq, kc = k < l ? k : l - 1;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        a[u][h] = fa(kc, h);
        b[u][h] = fb(kc, h);
      }
    }
    __builtin_amdgcn_sched_barrier(0);       // (all loads in flight before the first is waited for)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = 4 * (g + u) + kq < last;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        a[u][h] = in ? a[u][h] : (T)0;
        b[u][h] = in ? b[u][h] : (T)0;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = Mfma<T>::run(a[u][i], b[u][j], acc[i][j]);
    }
  }
  polish_sum<T>(acc, red, out);
}

// The same for the product of two sets of columns of M, which lie along k, in fp64 for either type: a lane reads four consecutive k at a
// time, one for each of four matrix instructions, and adds up the squares of what it has read (ni, nj).
template <typename T>
__device__ __forceinline__ void polish_gram(int l, const T *M, const int (&ic)[2], const int (&jc)[2], double *red, double (&out)[4],
                                            double (&ni)[2], double (&nj)[2]) {
  typedef T piece __attribute__((ext_vector_type(4), aligned(sizeof(T))));
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, kq = lane >> 4;
  const int groups = (l + 15) / 16, per = (groups + 3) / 4;
  const int g0 = wave * per, g1 = g0 + per < groups ? g0 + per : groups;
  f64x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = (f64x4)0.0;
  constexpr int U = sizeof(T) == 4 ? 4 : 2;
  for (int g = g0; g < g1; g += U) {
    piece a[U][2], b[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // (the last piece is read where it fits, l >= 4, and moved down below)
      const int k = 16 * (g + u) + 4 * kq, at = k + 4 <= l ? k : l - 4;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        a[u][h] = *reinterpret_cast<const piece *>(M + (int64_t)ic[h] * l + at);
        b[u][h] = *reinterpret_cast<const piece *>(M + (int64_t)jc[h] * l + at);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int left = g + u < g1 ? l - 16 * (g + u) - 4 * kq : 0, by = left >= 4 ? 0 : 4 - left;      // elements that exist; places to move
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        double x[2], y[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const T xv = by == 0 ? a[u][h][e] : by == 1 ? a[u][h][(e + 1) & 3] : by == 2 ? a[u][h][(e + 2) & 3] : a[u][h][(e + 3) & 3];
          const T yv = by == 0 ? b[u][h][e] : by == 1 ? b[u][h][(e + 1) & 3] : by == 2 ? b[u][h][(e + 2) & 3] : b[u][h][(e + 3) & 3];
          x[h] = e < left ? (double)xv : 0.0;
          y[h] = e < left ? (double)yv : 0.0;
          ni[h] = fma(x[h], x[h], ni[h]);
          nj[h] = fma(y[h], y[h], nj[h]);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = Mfma<double>::run(x[i], y[j], acc[i][j]);
      }
    }
  }
  polish_sum<double>(acc, red, out);
}

// Tile t of the tiles on or above the diagonal.
__device__ __forceinline__ void upper_tile(int tiles, int t, int &ti, int &tj) {
  ti = 0;
  while (t >= tiles - ti) { t -= tiles - ti; ++ti; }
  tj = ti + t;
}

enum { PO_ANGLES = 0, PO_SQUARE, PO_FOURTH, PO_PARTS, PO_EXP, PO_DOUBLE, PO_APPLY };

// Loads and stores that every XCD sees.
template <typename V> __device__ __forceinline__ V device_load(const V *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename V> __device__ __forceinline__ void device_store(V *p, V v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The device-wide stores of this wavefront have arrived where every XCD sees them (no write-back of the L2 is needed
// for those, which a release fence would ask for in every wavefront: 8 us a step more in fp64).
__device__ __forceinline__ void device_stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Waits until *p and *p2 reached `want`, or until *stop is set (if there is one); returns false in that case.
__device__ __forceinline__ bool jb_wait(const int *p, const int *p2, int want, const int *stop) {
  for (;;) {
    const int a = device_load(p), b = device_load(p2), st = stop != nullptr ? device_load(stop) : 0;
    if (a >= want && b >= want) return true;
    if (st != 0) return false;
    __builtin_amdgcn_s_sleep(1);
  }
}

// All corrections in one launch.  Tasks are the tiles of a phase, phase after phase; they are handed out by a counter, and a workgroup goes
// on to the next phase once every tile of the one before is finished.  As in jb_flow_kernel it waits for tasks with lower numbers only,
// whose workgroups are running, so no number of resident workgroups is assumed.  What a phase stores goes through to where every
// XCD sees it, and the wait ends by dropping what the caches of the reader hold.  The operands are l x l matrices, so a
// phase is a chain of latencies: counter, loads, sums, stores' arrival.
__device__ __forceinline__ void jb_wait_tiles(const int *p, int want) {
  while (device_load(p) < want) __builtin_amdgcn_s_sleep(4);
}

template <typename T>
__global__ __launch_bounds__(256) void polish_kernel(PolishParams<T> P) {
  JbSync *sync = P.sync;
  if (sync->run[0].stop != 2) return;
  const int l = P.l, tiles = P.tiles, upper = tiles * (tiles + 1) / 2;
  const T tol = Eps<T>::value * sqrt((T)l);
  const double floor2 = (double)Eps<T>::value * (double)Eps<T>::value * sync->fro2;
  __shared__ double red64[4 * kPoTile * kPoLd];
  T *red = reinterpret_cast<T *>(red64);
  __shared__ double part[4][2][kPoTile];
  __shared__ int ticket_sh;
  __shared__ float wave_rho[4], wave_x2[4], wave_open[4];
  T *M = P.b[0], *J = P.b[1], *X = P.b[2], *Y = P.b[3], *Y2 = P.b[4], *C = P.b[5], *S = P.b[6];
  int step = 0, phase = PO_ANGLES, seq = 0, base = 0, count = upper, order = 0, halvings = 0, doublings = 0, updates = 0;
  T half = (T)1;                                     // the series is taken of half * X
  float x_before = 1e30f, x_now = 0.f, x_all = 0.f, rho_now = 0.f;
  int ticket = 0;
  if (threadIdx.x == 0) ticket = atomicAdd(&sync->ticket, 1);

  for (;;) {
    if (threadIdx.x == 0) ticket_sh = ticket;
    __syncthreads();
    const int task = __builtin_amdgcn_readfirstlane(ticket_sh);
    // ---- the phase of this task
    while (task >= base + count) {
      if (threadIdx.x == 0) (void)jb_wait_tiles(&sync->done[seq], count);
      __syncthreads();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      base += count;
      ++seq;
      bool end = false, converged = false;
      if (phase == PO_ANGLES) {
        rho_now = __int_as_float(device_load(&sync->rho[step]));
        x_all = sqrtf((float)device_load(&sync->x2[step]) * (2.f / kPolishScale));
        x_now = sqrtf((float)device_load(&sync->x2_open[step]) * (2.f / kPolishScale));
        order = x_all <= polish_limit<T>(1) ? 1 : x_all <= polish_limit<T>(2) ? 2 : x_all <= polish_limit<T>(3) ? 3 : 4;
        converged = rho_now <= (float)tol;
        end = converged || !(x_now <= polish_start(l)) || !(x_now <= kPolishRate * x_before);
        halvings = 0;
        for (float x = x_all; x > polish_limit<T>(4) && halvings < 7; x *= 0.5f) ++halvings;
        doublings = halvings;
        half = ldexp((T)1, -halvings);
        phase = PO_SQUARE;
        count = upper;
      } else if (phase == PO_SQUARE && order >= 3) {
        phase = PO_FOURTH;
        count = upper;
      } else if (phase == PO_FOURTH && order >= 4) {
        phase = PO_PARTS;
        count = upper;
      } else if (phase < PO_EXP && order >= 2) {
        phase = PO_EXP;
        count = tiles * tiles;
      } else if ((phase == PO_EXP || phase == PO_DOUBLE) && doublings > 0) {
        if (phase == PO_DOUBLE) { T *t = C; C = S; S = t; }
        --doublings;
        phase = PO_DOUBLE;
        count = tiles * tiles;
      } else if (phase != PO_APPLY) {
        if (phase == PO_DOUBLE) { T *t = C; C = S; S = t; }              // (E is in C)
        phase = PO_APPLY;
        count = 2 * tiles * tiles;
      } else {
        // M and J are the new ones, what they were is free
        T *t = M; M = Y; Y = t;
        t = J; J = Y2; Y2 = t;
        ++updates;
        converged = rho_now * x_all <= (float)tol;             // the next one would find about that
        ++step;
        end = converged || step == kPolishSteps;
        x_before = x_now;
        phase = PO_ANGLES;
        count = upper;
      }
      if (end) {
        if (threadIdx.x == 0) {                                // (the same from every workgroup)
          device_store(&sync->updates, updates);
          device_store(&sync->converged, converged ? 1 : 0);
        }
        return;
      }
    }
    // ---- its tile
    if (threadIdx.x == 0) ticket = atomicAdd(&sync->ticket, 1);       // (the next one, in good time)
    int ti, tj;
    const int n = task - base, z = n >= tiles * tiles ? 1 : 0;
    const bool mirrored = phase <= PO_PARTS;               // symmetric or antisymmetric: tiles on or above the diagonal
    if (mirrored) upper_tile(tiles, n, ti, tj);
    else { ti = (n - z * tiles * tiles) / tiles; tj = (n - z * tiles * tiles) - ti * tiles; }
    const int i0 = ti * kPoTile, j0 = tj * kPoTile;
    // rows and columns beyond the last read the last one: what comes of them is not stored
    int ic[2], jc[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = i0 + 16 * h + (int)(threadIdx.x & 15), j = j0 + 16 * h + (int)(threadIdx.x & 15);
      ic[h] = i < l ? i : l - 1;
      jc[h] = j < l ? j : l - 1;
    }
    // the elements of this tile that its result needs besides the product, in flight with the operands
    T own[2][4];
    const T *own0 = phase == PO_APPLY ? (z == 0 ? M : J) : phase == PO_PARTS || (phase == PO_EXP && order < 4) ? Y : phase == PO_SQUARE ? X : C;
    const T *own1 = phase == PO_PARTS || (phase == PO_EXP && order == 3) ? Y2 : X;
    if (phase >= PO_PARTS || (phase == PO_SQUARE && order == 1)) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + 256 * u, i = i0 + (e >> 5), j = j0 + (e & 31);
        const int64_t at = (int64_t)(i < l ? i : l - 1) * l + (j < l ? j : l - 1);
        own[0][u] = own0[at];
        own[1][u] = own1[at];
      }
    }
    T v[4], w[4];
    auto store = [&](T *m, int i, int j, T a, T b) {
      device_store(m + (int64_t)i * l + j, a);
      if (mirrored && ti != tj) device_store(m + (int64_t)j * l + i, b);
    };
    auto each = [&](auto f) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + 256 * u, i = i0 + (e >> 5), j = j0 + (e & 31);
        if (i < l && j < l) f(u, i, j, (int64_t)i * l + j);
      }
    };
    auto at_i = [&](const T *m) { return [&, m](int k, int h) { return m[(int64_t)k * l + ic[h]]; }; };
    auto at_j = [&](const T *m) { return [&, m](int k, int h) { return m[(int64_t)k * l + jc[h]]; }; };
    auto minus_x = [&](int k, int h) { return -X[(int64_t)k * l + ic[h]]; };      // X[i][k]
    if (phase == PO_ANGLES) {
      double ni[2] = {0.0, 0.0}, nj[2] = {0.0, 0.0}, g[4];
      polish_gram<T>(l, M, ic, jc, red64, g, ni, nj);
      const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        ni[h] += __shfl_xor(ni[h], 16, 64); ni[h] += __shfl_xor(ni[h], 32, 64);
        nj[h] += __shfl_xor(nj[h], 16, 64); nj[h] += __shfl_xor(nj[h], 32, 64);
        if (lane < 16) { part[wave][0][16 * h + lane] = ni[h]; part[wave][1][16 * h + lane] = nj[h]; }
      }
      __syncthreads();
      float rho = 0.f, x2 = 0.f, open = 0.f;
      each([&](int u, int i, int j, int64_t) {
        if (ti == tj && i > j) return;
        const int r = i - i0, c = j - j0;
        const double di = (part[0][0][r] + part[1][0][r]) + (part[2][0][r] + part[3][0][r]);
        const double dj = (part[0][1][c] + part[1][1][c]) + (part[2][1][c] + part[3][1][c]);
        double angle = 0.0;
        if (i != j && di > floor2 && dj > floor2 && g[u] != 0.0) {
          const double rel = fabs(g[u]) / sqrt(di * dj);
          // tan of the angle as in rotation_params, then the angle itself (to the fifth order: it only has to be a good one)
          const double zeta = (dj - di) / (2.0 * g[u]), az = fabs(zeta);
          double t = az > 1e7 ? 0.5 / az : 1.0 / (az + sqrt(1.0 + zeta * zeta));
          t = zeta < 0.0 ? -t : t;
          // below the threshold only where it is a small one: inside a cluster it would be large, and noise
          if (rel > tol || fabs(t) <= kPolishFree) angle = t - t * t * t * (1.0 / 3.0 - 0.2 * t * t);
          if (rel > tol) {
            rho = fmaxf(rho, (float)rel);
            open += (float)(angle * angle);
          }
          x2 += (float)(angle * angle);
        }
        device_store(X + (int64_t)i * l + j, (T)angle);
        if (i != j) device_store(X + (int64_t)j * l + i, -(T)angle);
      });
#pragma unroll
      for (int m = 1; m < 64; m <<= 1) {
        rho = fmaxf(rho, __shfl_xor(rho, m, 64));
        x2 += __shfl_xor(x2, m, 64);
        open += __shfl_xor(open, m, 64);
      }
      if (lane == 0) { wave_rho[wave] = rho; wave_x2[wave] = x2; wave_open[wave] = open; }
      __syncthreads();
      if (threadIdx.x == 0) {
        rho = fmaxf(fmaxf(wave_rho[0], wave_rho[1]), fmaxf(wave_rho[2], wave_rho[3]));
        x2 = (wave_x2[0] + wave_x2[1]) + (wave_x2[2] + wave_x2[3]);
        open = (wave_open[0] + wave_open[1]) + (wave_open[2] + wave_open[3]);
        auto whole = [](float x) { return (unsigned long long)ceilf(fminf(x, 128.f) * kPolishScale); };
        if (x2 > 0.f) atomicAdd(&sync->x2[step], whole(x2));
        if (rho > 0.f) {
          atomicMax(&sync->rho[step], __float_as_int(rho));
          atomicAdd(&sync->x2_open[step], whole(open));
        }
      }
    } else if (phase == PO_SQUARE) {                 // Y = X X; with the shortest series E = X + Y / 2
      polish_tile<T>(l, minus_x, at_j(X), red, v);
      if (order == 1) {
        each([&](int u, int i, int j, int64_t) {
          const T x = own[0][u];
          store(C, i, j, x + (T)0.5 * v[u], (T)0.5 * v[u] - x);
        });
      } else {
        each([&](int u, int i, int j, int64_t) { store(Y, i, j, v[u], v[u]); });
      }
    } else if (phase == PO_FOURTH) {
      polish_tile<T>(l, at_i(Y), at_j(Y), red, v);
      each([&](int u, int i, int j, int64_t) { store(Y2, i, j, v[u], v[u]); });
    } else if (phase == PO_PARTS) {                  // Y^3, Y^4; cosine and sine part of half * X, without the I
      const T h2 = half * half, h4 = h2 * h2, h6 = h4 * h2, h8 = h4 * h4;
      polish_tile<T>(l, at_i(Y), at_j(Y2), red, v);
      polish_tile<T>(l, at_i(Y2), at_j(Y2), red, w);
      each([&](int u, int i, int j, int64_t) {
        const T y = h2 * own[0][u], y2 = h4 * own[1][u], y3 = h6 * v[u], y4 = h8 * w[u];
        const T c = ((y3 * (T)(1.0 / 720.0) + y4 * (T)(1.0 / 40320.0)) + y2 * (T)(1.0 / 24.0)) + y * (T)0.5;
        const T sn = ((y3 * (T)(1.0 / 5040.0) + y4 * (T)(1.0 / 362880.0)) + y2 * (T)(1.0 / 120.0)) + y * (T)(1.0 / 6.0);
        store(C, i, j, c, c);
        store(S, i, j, sn, sn);
      });
    } else if (phase == PO_EXP) {                    // E = cosine part + X + X (sine part)
      if (order == 4) {
        polish_tile<T>(l, minus_x, at_j(S), red, v);
        each([&](int u, int i, int j, int64_t) { store(C, i, j, (own[0][u] + half * v[u]) + half * own[1][u], (T)0); });
      } else if (order == 3) {
        polish_tile<T>(l, minus_x, [&](int k, int h) {
          const int64_t at = (int64_t)k * l + jc[h];
          return Y[at] * (T)(1.0 / 6.0) + Y2[at] * (T)(1.0 / 120.0);
        }, red, v);
        each([&](int u, int i, int j, int64_t at) {
          store(C, i, j, ((own[0][u] * (T)0.5 + own[1][u] * (T)(1.0 / 24.0)) + v[u]) + X[at], (T)0);
        });
      } else {
        polish_tile<T>(l, minus_x, [&](int k, int h) { return Y[(int64_t)k * l + jc[h]] * (T)(1.0 / 6.0); }, red, v);
        each([&](int u, int i, int j, int64_t) { store(C, i, j, (own[0][u] * (T)0.5 + v[u]) + own[1][u], (T)0); });
      }
    } else if (phase == PO_DOUBLE) {                 // exp(X)^2 - I = 2 E + E E, into S
      polish_tile<T>(l, [&](int k, int h) { return C[(int64_t)ic[h] * l + k]; }, at_j(C), red, v);
      each([&](int u, int i, int j, int64_t) { store(S, i, j, (T)2 * own[0][u] + v[u], (T)0); });
    } else {                                         // column i of the new matrix = that of the old one + sum_k E[k][i] column k
      const T *old = z == 0 ? M : J;
      T *next = z == 0 ? Y : Y2;
      polish_tile<T>(l, at_i(C), at_j(old), red, v);
      each([&](int u, int i, int j, int64_t) { store(next, i, j, own[0][u] + v[u], (T)0); });
    }
    device_stores_done();
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(&sync->done[seq], 1);
  }
}

template <typename T>
static void polish_launch(const rsvd_ctx *ctx, hipStream_t s, const PolishParams<T> &P) {
  int wgs = 2 * P.tiles * P.tiles;                   // tiles of the largest phase
  if (wgs > ctx->cu_count) wgs = ctx->cu_count;
  hipLaunchKernelGGL((polish_kernel<T>), dim3(wgs), dim3(256), 0, s, P);
}

// which: 0 = the sweeps from the start, until they have converged or (`corrections` follow) leave little enough for those; 1 = the
// sweeps behind the corrections, if those did not finish.  Mt2, Jt2: where an odd number of corrections has left M and J.
template <typename T>
__global__ __launch_bounds__(1024) void jb_flow_kernel(T *__restrict__ Mt, T *__restrict__ Jt, T *__restrict__ Mt2,
                                                       T *__restrict__ Jt2, int l, int nblk, int max_sweeps,
                                                       int *__restrict__ ver, JbSync *sync, int which, int corrections) {
  constexpr int b = kJgB;
  typedef typename Mfma<T>::vec acc_t;
  const T tol = Eps<T>::value * sqrt((T)l);
  const T floor2 = (T)(Eps<T>::value * Eps<T>::value * sync->fro2);
  JbRun *run = &sync->run[which];
  if (which != 0) {
    if (sync->run[0].stop != 2 || sync->converged != 0) return;
    if (sync->updates & 1) { Mt = Mt2; Jt = Jt2; }
    max_sweeps -= sync->run[0].used;
  }
  const int nblk2 = nblk + (nblk & 1), pairs = nblk2 / 2, steps_per_sweep = nblk2 - 1;
  const int ldp = jg_ldp<T>(l), lp = (l + 15) / 16 * 16;
  extern __shared__ __attribute__((aligned(16))) double lds_raw[];
  T *Pc = reinterpret_cast<T *>(lds_raw);                      // [2b][ldp]: column c of the panel, zero padded
  T *G0 = Pc + (size_t)kJgN * ldp;                             // G, even rounds
  T *R4 = G0 + kJgMat;                                         // four matrices: the five partial sums of G, then T, G1 (the third) and the (c, s) of every round
  double *Tm = reinterpret_cast<double *>(R4);                 // T[k][j], in the place of two of them in fp32, of one in fp64
  T *CS = R4 + 3 * kJgMat;                                     // [rounds][16 pairs][c, s]
  __shared__ int rotations, task;
  __shared__ unsigned turned;                                  // sum of s^2 over the rotations of the task, times kJbSumScale
  int ticket = 0;
  if (threadIdx.x == 0) ticket = atomicAdd(&run->ticket, 1);

  for (;;) {
    // (worked out anew for every task: the addresses that follow from them were kept across tasks otherwise, in
    // scratch memory)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, kq = lane >> 4;
    if (tid == 0) {
      bool go = ticket < max_sweeps * steps_per_sweep * pairs;
      if (go) {
        const int n = ticket / pairs, g = ticket - n * pairs;                  // step, pair
        const int sweep = n / steps_per_sweep, round = n - sweep * steps_per_sweep;
        if (round == 0) {
          if (sweep > 0) {
            const int *f = &run->finished[sweep - 1];
            go = jb_wait(f, f, steps_per_sweep * pairs, &run->stop);
            if (go) {
              const float rho = __int_as_float(device_load(&run->counters[sweep - 1]));
              const float before = sweep > 1 ? __int_as_float(device_load(&run->counters[sweep - 2])) : -1.f;
              const int stop = jacobi_done(rho, before, (float)tol)                                             ? 1
                               : corrections && sweeps_ready(device_load(&run->sumsq[sweep - 1]), rho, l) ? 2
                                                                                                                : 0;
              if (stop != 0) {
                device_store(&run->used, sweep);
                device_store(&run->stop, stop);
                go = false;
              }
            }
          }
        } else {
          const JbPair pr = jb_pair(1, round, g, l, b, nblk);
          go = jb_wait(ver + pr.bi, ver + (pr.valid ? pr.bj : pr.bi), n, &run->stop);
        }
      }
      task = go ? ticket : -1;
      rotations = 0;
      turned = 0u;
    }
    __syncthreads();
    if (task < 0) return;
    const int n = task / pairs, g = task - n * pairs;
    const int sweep = n / steps_per_sweep, round = n - sweep * steps_per_sweep;
    const JbPair pr = jb_pair(1, round, g, l, b, nblk);
    const int cols_i = pr.cols_i, cols_j = pr.cols_j;
    const int intra = (round == 0) ? b - 1 : 0;
    const int rounds = intra + (pr.valid ? b : 0);
    auto gcol = [&](int c) { return c < b ? pr.bi * b + c : pr.bj * b + (c - b); };      // global column of panel column c
    auto live = [&](int c) { return c < b ? c < cols_i : c - b < cols_j; };
    int rho_bits = 0;
    if (rounds > 0) {                                            // (a bye only passes its block on)
      // panel in: wavefront w takes columns w and w + 16, every load in flight before the first LDS store
      {
        constexpr int MAXJ = jg_max_order<T>() / 64;
        T v[2][MAXJ];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int c = wave + 16 * u;
          const T *src = Mt + (int64_t)gcol(live(c) ? c : 0) * l;
#pragma unroll
          for (int j = 0; j < MAXJ; ++j) {
            const int rr = lane + 64 * j;
            v[u][j] = (T)0;
            if (live(c) && rr < l) v[u][j] = device_load(src + rr);
          }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int c = wave + 16 * u;
#pragma unroll
          for (int j = 0; j < MAXJ; ++j) {
            const int rr = lane + 64 * j;
            if (rr < lp) Pc[c * ldp + rr] = v[u][j];
          }
        }
      }
      __syncthreads();

      // G = P^T P (symmetric: blocks (0,0), (0,1) and (1,1) only, five row slices each, fifteen wavefronts): a lane reads
      // 16 bytes down a column, which are the operands of two (fp64) or four matrix instructions, four such pieces ahead;
      // two accumulators
      {
        typedef T piece __attribute__((ext_vector_type(16 / sizeof(T))));
        constexpr int V = 16 / (int)sizeof(T);
        const int sl = wave / 3, tile = wave - 3 * sl;
        const int ti = tile >> 1, tj = (tile + 1) >> 1;
        const int steps = lp / (4 * V), per = (steps + 4) / 5;
        const int s0 = sl * per, s1 = (wave == 15) ? 0 : ((s0 + per < steps) ? s0 + per : steps);
        acc_t acc0 = (acc_t)(T)0, acc1 = (acc_t)(T)0;
        const piece *ap = reinterpret_cast<const piece *>(Pc + (ti * 16 + r16) * ldp + kq * V);
        const piece *bp = reinterpret_cast<const piece *>(Pc + (tj * 16 + r16) * ldp + kq * V);
        for (int st = s0; st < s1; st += 4) {
          piece av[4], bv[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            av[u] = (piece)(T)0;
            bv[u] = (piece)(T)0;
            if (st + u < s1) {
              av[u] = ap[4 * (st + u)];
              bv[u] = bp[4 * (st + u)];
            }
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (st + u < s1) {
#pragma unroll
              for (int x = 0; x < V; x += 2) {
                acc0 = Mfma<T>::run(av[u][x], bv[u][x], acc0);
                acc1 = Mfma<T>::run(av[u][x + 1], bv[u][x + 1], acc1);
              }
            }
        }
        if (wave < 15) {
          T *dst = R4 + sl * kJgPart + tile * 256;
#pragma unroll
          for (int v = 0; v < 4; ++v) dst[Mfma<T>::row(lane, v) * 16 + r16] = acc0[v] + acc1[v];
        }
      }
      __syncthreads();
      {
        // entry (i, j) of G from the five partial sums of its block (the block above the diagonal read transposed below it)
        const int i = tid >> 5, j = tid & 31;
        const int bi2 = i >> 4, bj2 = j >> 4;
        const bool lower = bi2 > bj2;
        const int tile = lower ? 1 : bi2 + bj2;
        const int e = tile * 256 + (lower ? (j & 15) * 16 + (i & 15) : (i & 15) * 16 + (j & 15));
        G0[i * kJgLd + j] =
            ((R4[e] + R4[kJgPart + e]) + (R4[2 * kJgPart + e] + R4[3 * kJgPart + e])) + R4[4 * kJgPart + e];
      }
      __syncthreads();
      // The rounds.  Wavefronts 0-3 (one per SIMD; what bounds a round is the number of instructions they issue, one every
      // four cycles): G <- J^T G J, thread (a, bb) the rows of pair a and the columns of pair bb; every lane works out the
      // rotation of pair bb, and the first sixteen leave (c, s) of the round in LDS.  Wavefronts 4-11: T <- T J one round
      // behind, in fp64, thread (rr, bb) row rr and the columns of pair bb.  One barrier per round (G alternates between two
      // copies; the two elements of T that a thread changes are its own in that round).
      float rho = 0.f, s2 = 0.f;
      auto run_rounds = [&](auto kind, int r0, int count) {        // rounds r0, ... of the task
        constexpr bool INTRA = decltype(kind)::value;
        if (wave < 4) {
          // lane 0 of a row of 16 lanes holds pair bb = a, whose rotation it hands to the others
          const int a = tid >> 4, bb = (tid + a) & 15;
          int pa, qa, mpa, mqa, pb, qb, mpb, mqb;
          jg_pair<INTRA>(a, pa, qa, mpa, mqa);
          jg_pair<INTRA>(bb, pb, qb, mpb, mqb);
          T *cs = CS + bb * 2;
          for (int r = 0; r < count; ++r) {
            const int odd = (r0 + r) & 1;                          // (offsets: a choice between pointers into LDS makes flat accesses)
            const T *Gs = G0 + odd * (3 * kJgMat);
            T *Gd = G0 + (odd ^ 1) * (3 * kJgMat);
            T cb, sb;
            const T g00 = Gs[pa * kJgLd + pb], g01 = Gs[pa * kJgLd + qb];
            const T g10 = Gs[qa * kJgLd + pb], g11 = Gs[qa * kJgLd + qb];
            const float rel = jg_pair_params<T>(Gs, pb, qb, tol, floor2, cb, sb);
            const T ca = dpp_mov<0x150>(cb), sa = dpp_mov<0x150>(sb);          // row_newbcast:0
            const T h00 = ca * g00 - sa * g10, h01 = ca * g01 - sa * g11;
            const T h10 = sa * g00 + ca * g10, h11 = sa * g01 + ca * g11;
            T n00 = cb * h00 - sb * h01, n01 = sb * h00 + cb * h01;
            T n10 = cb * h10 - sb * h11, n11 = sb * h10 + cb * h11;
            if (a == bb && rel > 0.f) {
              n01 = (T)0;
              n10 = (T)0;
              rho = fmaxf(rho, rel);
              s2 += (float)(sb * sb);
            }
            Gd[mpa * kJgLd + mpb] = n00; Gd[mpa * kJgLd + mqb] = n01;
            Gd[mqa * kJgLd + mpb] = n10; Gd[mqa * kJgLd + mqb] = n11;
            if (a == 0) {
              cs[r * 32] = cb;
              cs[r * 32 + 1] = sb;
            }
            __syncthreads();
          }
          __syncthreads();
        } else {
          const int rr = (tid - 256) >> 4, bb = tid & 15;
          const T *cs = CS + bb * 2;
          double *Tr = Tm + rr * kJgLd;
          for (int r = -1; r < count; ++r) {                       // T <- T J_r, one round behind
            if (r >= 0 && wave < 12) {
              int pb, qb;
              jg_columns<INTRA>(bb, r, pb, qb);
              double cb = (double)cs[r * 32], sb = (double)cs[r * 32 + 1];
              if (sizeof(T) == 4) {
                // (c, s) of the fp32 instructions is off length 1 by up to 1e-7, to one side for small angles
                const double off = 0.5 * fma(sb, sb, fma(cb, cb, -1.0));
                cb -= cb * off;
                sb -= sb * off;
              }
              double tp = Tr[pb], tq = Tr[qb];
              if (r0 + r == 0) {                                   // (T is the identity)
                tp = rr == pb ? 1.0 : 0.0;
                tq = rr == qb ? 1.0 : 0.0;
              }
              Tr[pb] = cb * tp - sb * tq;
              Tr[qb] = sb * tp + cb * tq;
            }
            __syncthreads();
          }
        }
      };
      if (round == 0) run_rounds(JbKind<true>(), 0, intra);
      if (pr.valid) run_rounds(JbKind<false>(), intra, b);
      if (rho > 0.f) {
        atomicMax(&rotations, __float_as_int(rho));
        atomicAdd(&turned, (unsigned)ceilf(s2 * kJbSumScale));             // (whole numbers: the sum does not depend on the order)
      }
      __syncthreads();
      rho_bits = rotations;
    }

    if (rho_bits != 0) {
      // panel out: (P T)^T = T^T P^T in 16 x 16 blocks; wavefront w takes the output columns jb * 16 ... and the row
      // blocks rb, rb + 8, ..., two of them at a time
      const int jb = wave & 1;
      T ta[kJgN / 4];
#pragma unroll
      for (int ks = 0; ks < kJgN / 4; ++ks) ta[ks] = (T)Tm[(4 * ks + kq) * kJgLd + jb * 16 + r16];     // A[i = column][k] = T[k][column]
      const int nrb = lp / 16;
      for (int rb = wave >> 1; rb < nrb; rb += 16) {
        const int rb2 = rb + 8;
        const bool two = rb2 < nrb;
        const T *bp0 = Pc + kq * ldp + rb * 16 + r16;                                              // B[k][n = row] = P[row][k]
        const T *bp1 = Pc + kq * ldp + (two ? rb2 : rb) * 16 + r16;
        T b0[kJgN / 4], b1[kJgN / 4];
#pragma unroll
        for (int ks = 0; ks < kJgN / 4; ++ks) { b0[ks] = bp0[(4 * ks) * ldp]; b1[ks] = bp1[(4 * ks) * ldp]; }
        acc_t acc0 = (acc_t)(T)0, acc1 = (acc_t)(T)0;
#pragma unroll
        for (int ks = 0; ks < kJgN / 4; ++ks) {
          acc0 = Mfma<T>::run(ta[ks], b0[ks], acc0);
          acc1 = Mfma<T>::run(ta[ks], b1[ks], acc1);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int c = jb * 16 + Mfma<T>::row(lane, v);
          if (live(c)) {
            T *dst = Mt + (int64_t)gcol(c) * l;
            if (rb * 16 + r16 < l) device_store(dst + rb * 16 + r16, acc0[v]);
            if (two && rb2 * 16 + r16 < l) device_store(dst + rb2 * 16 + r16, acc1[v]);
          }
        }
      }
    }
    device_stores_done();
    __syncthreads();
    if (tid == 0) {
      device_store(ver + pr.bi, n + 1);
      if (pr.valid) device_store(ver + pr.bj, n + 1);
      if (rho_bits != 0) {
        atomicMax(&run->counters[sweep], rho_bits);
        atomicAdd(&run->sumsq[sweep], (unsigned long long)turned);
      }
      device_stores_done();                                      // (counters before finished)
      atomicAdd(&run->finished[sweep], 1);
      ticket = atomicAdd(&run->ticket, 1);
      // J: the same two blocks of columns, after the step before
      int *verj = ver + nblk;
      (void)jb_wait(verj + pr.bi, verj + (pr.valid ? pr.bj : pr.bi), n, nullptr);
    }
    __syncthreads();
    if (rho_bits != 0) {
      // wavefront w takes the row blocks w, w + 16, ...: it reads both blocks of columns before it writes either
      T ta[2][kJgN / 4];
#pragma unroll
      for (int ks = 0; ks < kJgN / 4; ++ks) {
        ta[0][ks] = (T)Tm[(4 * ks + kq) * kJgLd + r16];
        ta[1][ks] = (T)Tm[(4 * ks + kq) * kJgLd + 16 + r16];
      }
      for (int rb = wave; rb < lp / 16; rb += 16) {
        const int row = rb * 16 + r16;
        T bv[kJgN / 4];
#pragma unroll
        for (int ks = 0; ks < kJgN / 4; ++ks) {
          const int c = 4 * ks + kq;
          bv[ks] = (T)0;
          if (live(c) && row < l) bv[ks] = device_load(Jt + (int64_t)gcol(c) * l + row);
        }
        acc_t acc[2] = {(acc_t)(T)0, (acc_t)(T)0};
#pragma unroll
        for (int ks = 0; ks < kJgN / 4; ++ks) {
          acc[0] = Mfma<T>::run(ta[0][ks], bv[ks], acc[0]);
          acc[1] = Mfma<T>::run(ta[1][ks], bv[ks], acc[1]);
        }
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int c = jb * 16 + Mfma<T>::row(lane, v);
            if (live(c) && row < l) device_store(Jt + (int64_t)gcol(c) * l + row, acc[jb][v]);
          }
      }
    }
    device_stores_done();
    __syncthreads();
    if (tid == 0) {
      device_store(ver + nblk + pr.bi, n + 1);
      if (pr.valid) device_store(ver + nblk + pr.bj, n + 1);
    }
  }
}

// Column norms (one wavefront per column), then ranks by counting, then the scatter.
template <typename T>
__global__ __launch_bounds__(256) void jb_norms_kernel(const T *__restrict__ Mt, const T *__restrict__ Mt2, int l,
                                                       T *__restrict__ nrm, const JbSync *sync) {
  if (sync != nullptr && (sync->updates & 1)) Mt = Mt2;
  const int col = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (col >= l) return;
  T s2 = 0;
  for (int r = lane; r < l; r += 64) { const T x = Mt[(int64_t)col * l + r]; s2 += x * x; }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s2 += __shfl_xor(s2, off, 64);
  if (lane == 0) nrm[col] = sqrt(s2);
}

template <typename T>
__global__ __launch_bounds__(256) void jb_rank_kernel(const T *__restrict__ nrm, int l, int *__restrict__ rnk,
                                                      SigmaOut sig, const JbHeader *hdr, int max_sweeps,
                                                      DevInfo *info, const JbSync *sync) {
  // sixteen threads to a column, each compares it with a sixteenth of the others (one thread for all of them: 17 us at l = 210, 35 at 450)
  const int sub = threadIdx.x & 15, j = blockIdx.x * 16 + (threadIdx.x >> 4);
  const T mine = nrm[j < l ? j : 0];
  int rank = 0;
#pragma unroll 8
  for (int i = sub; i < l; i += 16) {
    const T o = nrm[i];
    rank += (o > mine || (o == mine && i < j)) ? 1 : 0;
  }
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) rank += __shfl_xor(rank, m, 16);
  if (j < l && sub == 0) {
    rnk[j] = rank;
    if (rank < sig.n) reinterpret_cast<T *>(sig.p)[rank] = mine * (T)hdr->unscale;
  }
  if (j == 0 && sub == 0 && info != nullptr) {
    const float tol = (float)(Eps<T>::value * sqrt((T)l));
    int used = max_sweeps;
    bool done;
    if (sync != nullptr) {
      // a run that stopped says why; one that did not went on to the limit, with its last sweep yet to be looked at
      const JbRun &first = sync->run[0], &second = sync->run[1];
      if (first.stop == 2) {
        const int left = max_sweeps - first.used;
        used = first.used + sync->updates + (sync->converged ? 0 : second.stop != 0 ? second.used : left);
        done = sync->converged || second.stop != 0 || jacobi_done_before(second.counters, left, tol);
      } else {
        if (first.stop != 0) used = first.used;
        done = first.stop != 0 || jacobi_done_before(first.counters, max_sweeps, tol);
      }
    } else {
      for (int s = 1; s <= max_sweeps; ++s)
        if (jacobi_done_before(hdr->counters, s, tol)) { used = s; break; }
      done = jacobi_done_before(hdr->counters, max_sweeps, tol);
    }
    atomicMax(&info->jacobi_sweeps, used);
    if (!done) atomicMax(&info->status, (int)RSVD_ERR_NO_CONVERGENCE);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void jb_scatter_kernel(const T *__restrict__ Mt, const T *__restrict__ Jt,
                                                         const T *__restrict__ Mt2, const T *__restrict__ Jt2, int l,
                                                         const T *__restrict__ nrm, const int *__restrict__ rnk,
                                                         const JbHeader *hdr, T *__restrict__ X, T *__restrict__ W,
                                                         const JbSync *sync) {
  if (sync != nullptr && (sync->updates & 1)) { Mt = Mt2; Jt = Jt2; }
  const T floor2 = (T)(Eps<T>::value * Eps<T>::value * hdr->fro2);
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < (int64_t)l * l;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(idx / l), r = (int)(idx - (int64_t)c * l);
    const T s = nrm[c];
    const int64_t dst = (int64_t)r * l + rnk[c];
    X[dst] = (s * s > floor2) ? Mt[idx] / s : (T)0;
    W[dst] = Jt[idx];
  }
}

constexpr int kJbMaxSweeps = 24;           // of jb_panel_kernel, whose every sweep is launched

// Lanes per column pair of the LDS-resident kernel.
static int jacobi_group(rsvd_dtype dtype, int64_t l) {
  (void)dtype; (void)l;
  return 16;       // measured: 16 beats 8 from l = 20 to 128 (a round is one wavefront's dependent chain), 4 is slowest
}

static size_t jacobi_lds_bytes(rsvd_dtype dtype, int64_t l) {
  const size_t es = dtype_size(dtype);
  const size_t ldm = (size_t)jacobi_ldm((int)l, jacobi_group(dtype, l), (int)es);
  return align_up(2 * (size_t)l * ldm * es + (size_t)l * (es + sizeof(int)), 16);
}

int jacobi_max_lds_order(const rsvd_ctx *ctx, rsvd_dtype dtype) {
  int l = 2;
  while (l < 128 && jacobi_lds_bytes(dtype, l + 1) + 4096 <= ctx->lds_per_block) ++l;
  return l;      // 128 columns = 64 pairs x 16 lanes = the largest workgroup
}

// Largest order of a batched call: fp64 orders beyond the LDS-resident kernel keep J in global memory, up to the
// largest workgroup (64 pairs x 16 lanes).
int jacobi_max_batched_order(const rsvd_ctx *ctx, rsvd_dtype dtype) {
  return dtype == RSVD_F64 ? 128 : jacobi_max_lds_order(ctx, dtype);
}
static size_t jacobi_jglobal_bytes(int64_t l) {
  return (size_t)l * (size_t)jacobi_ldm((int)l, 16, 8) * 8;
}

// Units (8 bytes) per lane for order l: ceil(l / V / 32), rounded up to one of these values; kernels exist for those of orders beyond
// the flow kernel (16 and more in fp64, 18 and more in fp32), from the others follows the block width only.
static int jb_units_per_lane(rsvd_dtype dtype, int64_t l) {
  const int v = 8 / (int)dtype_size(dtype);
  const int need = (int)ceil_div(ceil_div(l, v), 32);
  static const int avail[] = {2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 14, 16, 18, 20, 24};
  for (int a : avail)
    if (a >= need) return a;
  return 0;
}

// block width for the panel kernel: b padded columns plus the 2b x 2b T must fit in LDS
static int jb_block_width(const rsvd_ctx *ctx, rsvd_dtype dtype, int64_t l) {
  const size_t es = dtype_size(dtype);
  const int nv = jb_units_per_lane(dtype, l);
  if (nv == 0) return 0;
  const size_t ldp = (size_t)32 * nv * (8 / es) + 2;
  // Measured from l = 130 to 576 in both precisions: 16 beats 24 and 32 (a round is bound by instruction issue,
  // so fewer wavefronts per SIMD make it shorter, which outweighs the larger number of launches), 8 is slower.
  for (int b = 16; b >= 8; b -= 8) {
    const size_t need = ((size_t)b * ldp + (size_t)(2 * b) * (2 * b + 2)) * es + 1024;   // one block of columns + T
    if (need <= ctx->lds_per_block) return b;
  }
  return 0;
}

// One workgroup that rotates columns in LDS, or many on blocks of columns with corrections behind (us; triangular factors of a Gaussian
// matrix, and of nearly aligned factors with values exp(-3 i / l) and (1 + i)^-1/2):
//   fp32  l = 80 448, 217, 218 against 488, 228, 269; 96 534, 260, 258 against 486, 249, 273; 104 740, 336, 342 against 652, 290, 332;
//         120 796, 396, 399 against 662, 300, 354 (100000 x 1000 centred, l = 120, q = 3: 2898 -> 2715 for the whole call)
//   fp64  l = 56 395, 239, 242 against 429, 245, 269; 64 479, 266, 275 against 393, 245, 271; 72 700, 409, 414 against 592, 296, 325;
//         96 1064, 571, 583 against 582, 303, 365
// In fp32 the line lies where all three are faster (at 96 one is not).  In fp64 the blocks win at 64 already, and lose at 56; the orders between
// are not measured, and the line is the first order behind them.  Factors with many equal values, which the corrections leave to sweeps, gain
// less: l = 98 with 90 of them, 45 matrices, fp64 1318 -> 1306, fp32 514 -> 629.  (The one workgroup of these figures had no corrections; up to l = 80
// and 64 it has them by now and takes less, see lds_takes_corrections.)
bool jacobi_prefers_blocks(rsvd_dtype dtype, int64_t l) { return l >= (dtype == RSVD_F32 ? 97 : 65); }

// Scratch of the block path: header, Mt, Jt, norms, ranks.
size_t jacobi_scratch_bytes(const rsvd_ctx *ctx, rsvd_dtype dtype, int64_t l) {
  if (l <= jacobi_max_lds_order(ctx, dtype)) return 0;
  if (jb_block_width(ctx, dtype, l) == 0) return 0;          // unsupported order
  const size_t es = dtype_size(dtype);
  const size_t b = (size_t)jb_block_width(ctx, dtype, l), nblk = ceil_div((size_t)l, b);
  return align_up(sizeof(JbHeader), 256) + 2 * align_up((size_t)l * l * es, 256) + align_up((size_t)l * es, 256) +
         align_up((size_t)l * sizeof(int), 256) + align_up(2 * nblk * 4 * b * b * es, 256) +
         align_up(2 * nblk * sizeof(int), 256);
}

// The flow kernel is written for 16 columns to a block and holds the panel of a block pair in LDS; longer columns
// are rotated in place by the panel kernel.
template <typename T>
static bool jb_takes_flow(const rsvd_ctx *ctx, int b, int l) {
  return b == kJgB && l <= jg_max_order<T>() && jg_lds_bytes<T>(l) <= kJgLds && kJgLds + 1024 <= ctx->lds_per_block;
}

template <typename T>
static hipError_t jacobi_block_launch(rsvd_ctx *ctx, hipStream_t s, rsvd_dtype dtype, int l, const double *M,
                                      SigmaOut sig, T *X, T *W, DevInfo *info, char *scratch, int rows,
                                      const JacobiSlots *slots) {
  const int b = jb_block_width(ctx, dtype, l);
  if (b == 0) return hipErrorNotSupported;
  const size_t es = sizeof(T);
  const int nblk = (l + b - 1) / b;
  // (orders that the workspace has no scratch for work in the slots: M and J in the first two, all but the matrices in the last)
  const bool in_slots = l <= jacobi_max_lds_order(ctx, dtype);
  char *p = in_slots ? (char *)slots->slot[7] : scratch;
  auto take = [&](size_t bytes) { char *at = p; p += align_up(bytes, 256); return at; };
  JbHeader *hdr = reinterpret_cast<JbHeader *>(take(sizeof(JbHeader)));
  T *Mt = in_slots ? (T *)slots->slot[0] : reinterpret_cast<T *>(take((size_t)l * l * es));
  T *Jt = in_slots ? (T *)slots->slot[1] : reinterpret_cast<T *>(take((size_t)l * l * es));
  T *nrm = reinterpret_cast<T *>(take((size_t)l * es));
  int *rnk = reinterpret_cast<int *>(take((size_t)l * sizeof(int)));
  // [2][nblk][2b][2b]; the flow kernel has no use for it: its counters lie there
  T *Tring = reinterpret_cast<T *>(take(in_slots ? sizeof(JbSync) + (size_t)2 * nblk * sizeof(int) : (size_t)2 * nblk * 4 * b * b * es));
  int *chg = reinterpret_cast<int *>(p);                                                        // [2][nblk]
  const int nblk2 = nblk + (nblk & 1);
  const int nv = jb_units_per_lane(dtype, l);
  const size_t ldp = (size_t)32 * nv * (8 / es) + 2;
  const size_t lds_rot = ((size_t)b * ldp + (size_t)(2 * b) * (2 * b + 2)) * es;
  const size_t lds_j = ((size_t)(2 * b) * (kJbRowChunk + 8) + (size_t)(2 * b) * (2 * b + 2)) * es;   // jb_apply_t
  const size_t lds = lds_rot > lds_j ? lds_rot : lds_j;
  const int chunks = (l + kJbRowChunk - 1) / kJbRowChunk;
  const bool flow = jb_takes_flow<T>(ctx, b, l);
  JbSync *sync = flow ? reinterpret_cast<JbSync *>(Tring) : nullptr;
  int *ver2 = reinterpret_cast<int *>(sync + 1);
  ProfScope ps(ctx, s, PK_JACOBI);
  hipLaunchKernelGGL(jb_fro_kernel, dim3(kJbFroParts), dim3(256), 0, s, M, l, hdr);
  {
    int64_t blocks = ((int64_t)l * l + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL((jb_init_kernel<T>), dim3((unsigned)blocks), dim3(256), 0, s, M, l, Mt, Jt, hdr, rows, chg,
                       2 * nblk, sync, ver2);
  }
  T *Mt2 = Mt, *Jt2 = Jt;
  if (flow) {
    const int corrections = slots != nullptr ? 1 : 0;
    if (corrections) {
      PolishParams<T> P;
      P.b[0] = Mt; P.b[1] = Jt;
      for (int i = 0; i < 5; ++i) P.b[2 + i] = (T *)slots->slot[i + (in_slots ? 2 : 0)];
      Mt2 = P.b[3]; Jt2 = P.b[4];
      P.sync = sync; P.l = l; P.tiles = (l + kPoTile - 1) / kPoTile;
      hipLaunchKernelGGL((jb_flow_kernel<T>), dim3(nblk2), dim3(1024), jg_lds_bytes<T>(l), s, Mt, Jt, Mt2, Jt2, l, nblk,
                         kJacobiMaxSweeps, chg, sync, 0, 1);
      polish_launch<T>(ctx, s, P);
    }
    hipLaunchKernelGGL((jb_flow_kernel<T>), dim3(nblk2), dim3(1024), jg_lds_bytes<T>(l), s, Mt, Jt, Mt2, Jt2, l, nblk,
                       kJacobiMaxSweeps, corrections ? ver2 : chg, sync, corrections, 0);
  } else {
#define RSVD_JB_CASE(NVV)                                                                                        \
  case NVV: {                                                                                                    \
    int slot = 0, pp = -1, pr = 0, psw = 0, pwgs = 0;          /* the launch before: phase, round, sweep, pairs */ \
    auto go = [&](int phase, int round, int sweep, int wgs) {                                                    \
      hipLaunchKernelGGL((jb_panel_kernel<T, NVV>), dim3(wgs + pwgs * chunks), dim3(1024), lds, s, Mt, Jt, l,    \
                         b, nblk, phase, round, sweep, wgs, pp, pr, psw, Tring, chg, slot, hdr);                 \
      pp = phase; pr = round; psw = sweep; pwgs = wgs; slot ^= 1;                                                \
    };                                                                                                           \
    for (int sweep = 0; sweep < kJbMaxSweeps; ++sweep) {                                                         \
      go(0, 0, sweep, nblk);                                                                                     \
      for (int round = 0; round < nblk2 - 1; ++round) go(1, round, sweep, nblk2 / 2);                            \
    }                                                                                                            \
    go(0, 0, kJbMaxSweeps, 0);                                 /* applies the T of the last round */            \
  } break
    switch (nv) {                                              // (smaller orders take the flow kernel)
      RSVD_JB_CASE(18); RSVD_JB_CASE(20); RSVD_JB_CASE(24);
      default:
        if constexpr (sizeof(T) == 8) {
          switch (nv) {
            RSVD_JB_CASE(16);
            default: return hipErrorNotSupported;
          }
        } else {
          return hipErrorNotSupported;
        }
    }
#undef RSVD_JB_CASE
  }
  hipLaunchKernelGGL((jb_norms_kernel<T>), dim3((l + 3) / 4), dim3(256), 0, s, Mt, Mt2, l, nrm, sync);
  hipLaunchKernelGGL((jb_rank_kernel<T>), dim3((l + 15) / 16), dim3(256), 0, s, nrm, l, rnk, sig, hdr,
                     flow ? kJacobiMaxSweeps : kJbMaxSweeps, info, sync);
  hipLaunchKernelGGL((jb_scatter_kernel<T>), dim3(256), dim3(256), 0, s, Mt, Jt, Mt2, Jt2, l, nrm, rnk, hdr, X, W, sync);
  return hipGetLastError();
}

// (The corrections have kernels of their own: with them a kernel takes 99 to 128 registers, without 32 to 72, and twice as many
// wavefronts of it fit a CU.)
template <typename T, typename TIn, int RPL, int G>
static hipError_t launch_lds(hipStream_t s, int nt, size_t lds, const void *M, int l, const SigmaOut &sig, void *X, void *W,
                             DevInfo *info, int batch, int64_t stride, int rows, bool corrections) {
  if constexpr (CorrCfg<T, RPL>::kFits) {
    if (corrections) {
      hipLaunchKernelGGL((jacobi_lds_kernel<T, TIn, RPL, G, false, true>), dim3(batch), dim3(nt), lds, s, (const TIn *)M, l,
                         sig, (T *)X, (T *)W, info, stride, rows, (T *)nullptr);
      return hipGetLastError();
    }
  }
  if (corrections) return hipErrorInvalidValue;
  hipLaunchKernelGGL((jacobi_lds_kernel<T, TIn, RPL, G>), dim3(batch), dim3(nt), lds, s, (const TIn *)M, l,
                     sig, (T *)X, (T *)W, info, stride, rows, (T *)nullptr);
  return hipGetLastError();
}
// fp64 orders 97 .. 128: M in LDS, J in global memory
template <int RPL>
static hipError_t launch_lds_jg(hipStream_t s, int nt, size_t lds, const void *M, int l, const SigmaOut &sig, void *X, void *W,
                                DevInfo *info, int batch, int64_t stride, int rows, void *Jglobal) {
  hipLaunchKernelGGL((jacobi_lds_kernel<double, double, RPL, 16, true>), dim3(batch), dim3(nt), lds, s,
                     (const double *)M, l, sig, (double *)X, (double *)W, info, stride, rows,
                     (double *)Jglobal);
  return hipGetLastError();
}

// rows per lane = padded rows / G
template <typename T, typename TIn>
static hipError_t launch_lds_g(hipStream_t s, int nt, int G, int rpl, size_t lds, const void *M, int l, const SigmaOut &sig,
                               void *X, void *W, DevInfo *info, int batch, int64_t stride, int rows, bool corrections) {
  if (G == 16) {
    // fp32 rows come in pairs (8-byte units), fp64 rows singly
    if constexpr (sizeof(T) == 8) {
      switch (rpl) {
        case 1: return launch_lds<T, TIn, 1, 16>(s, nt, lds, M, l, sig, X, W, info, batch, stride, rows, corrections);
        case 3: return launch_lds<T, TIn, 3, 16>(s, nt, lds, M, l, sig, X, W, info, batch, stride, rows, corrections);
        case 5: return launch_lds<T, TIn, 5, 16>(s, nt, lds, M, l, sig, X, W, info, batch, stride, rows, corrections);
        default: break;
      }
    }
    switch (rpl) {
      case 2: return launch_lds<T, TIn, 2, 16>(s, nt, lds, M, l, sig, X, W, info, batch, stride, rows, corrections);
      case 4: return launch_lds<T, TIn, 4, 16>(s, nt, lds, M, l, sig, X, W, info, batch, stride, rows, corrections);
      case 6: return launch_lds<T, TIn, 6, 16>(s, nt, lds, M, l, sig, X, W, info, batch, stride, rows, corrections);
      case 8: return launch_lds<T, TIn, 8, 16>(s, nt, lds, M, l, sig, X, W, info, batch, stride, rows, corrections);
      default: return hipErrorNotSupported;
    }
  }
  return hipErrorNotSupported;
}

// The two matrices that the corrections work in.
static size_t corr_lds_bytes(rsvd_dtype dtype, int64_t l) {
  return 2 * (size_t)(ceil_div(l, 16) * 16) * (size_t)corr_ld((int)l) * dtype_size(dtype);
}

// The kernels of this file are launched with up to 156 KB of dynamic LDS (jb_flow_kernel: kJgLds): the limit is raised here, once per
// context (with its device current), for every instantiation the dispatch above can reach and whose largest order asks for more than
// the default of 64 KB (each call takes 3 to 4 us of rsvd_create).
template <typename T, typename TIn, int RPL>
static void raise_lds_limit_lds(hipError_t &e) {
  constexpr rsvd_dtype dtype = sizeof(T) == 4 ? RSVD_F32 : RSVD_F64;
  const size_t bytes = jacobi_lds_bytes(dtype, 16 * RPL);
  if (e == hipSuccess && bytes > 60 * 1024)
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&jacobi_lds_kernel<T, TIn, RPL, 16>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 4096);
  if constexpr (CorrCfg<T, RPL>::kFits) {
    const int64_t l = 16 * RPL < corr_max_order(sizeof(T) == 4) ? 16 * RPL : corr_max_order(sizeof(T) == 4);
    if (e == hipSuccess && jacobi_lds_bytes(dtype, l) + corr_lds_bytes(dtype, l) > 60 * 1024)
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(&jacobi_lds_kernel<T, TIn, RPL, 16, false, true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 4096);
  }
}
template <int RPL>
static void raise_lds_limit_jg(hipError_t &e) {
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&jacobi_lds_kernel<double, double, RPL, 16, true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 4096);
}
template <typename T, int NV>
static void raise_lds_limit_panel(hipError_t &e) {
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&jb_panel_kernel<T, NV>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 4096);
}
template <typename T>
static void raise_lds_limit_panels(hipError_t &e) {
  if constexpr (sizeof(T) == 8) raise_lds_limit_panel<T, 16>(e);
  raise_lds_limit_panel<T, 18>(e); raise_lds_limit_panel<T, 20>(e); raise_lds_limit_panel<T, 24>(e);
}

hipError_t jacobi_init_device(rsvd_ctx *ctx) {
  (void)ctx;
  hipError_t e = hipSuccess;
  raise_lds_limit_lds<float, double, 2>(e); raise_lds_limit_lds<float, double, 4>(e);
  raise_lds_limit_lds<float, double, 6>(e); raise_lds_limit_lds<float, double, 8>(e);
  raise_lds_limit_lds<float, float, 2>(e); raise_lds_limit_lds<float, float, 4>(e);
  raise_lds_limit_lds<float, float, 6>(e); raise_lds_limit_lds<float, float, 8>(e);
  raise_lds_limit_lds<double, double, 1>(e); raise_lds_limit_lds<double, double, 2>(e);
  raise_lds_limit_lds<double, double, 3>(e); raise_lds_limit_lds<double, double, 4>(e);
  raise_lds_limit_lds<double, double, 5>(e); raise_lds_limit_lds<double, double, 6>(e);
  raise_lds_limit_lds<double, double, 8>(e);
  raise_lds_limit_jg<7>(e);
  raise_lds_limit_jg<8>(e);
  raise_lds_limit_panels<float>(e);
  raise_lds_limit_panels<double>(e);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&jb_flow_kernel<float>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kJgLds);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&jb_flow_kernel<double>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kJgLds);
  return e;
}

// From 16 columns on (12: 44 -> 49 us; in fp32 below 24 it depends on the values whether the corrections bring more than a sweep of this kernel takes longer:
// 300 x 200, l = 16, values that fall by e^-0.25 each 40 -> 36, low rank and noise 41 -> 43), and where no CU has two problems of a batch: with up to 16
// wavefronts, twice the registers and twice the LDS a problem they no longer run side by side (fp32, q = 2, us without and with: 1500 x (l = 24)
// 89, 233; 600 x 48 223, 262; 300 x 72 369, 419; 300 x 80 450, 484; 256 x 48 128, 99; fp64 600 x 40 369, 402; 300 x 64 550, 492; 256 x 64 377, 274).
static bool lds_takes_corrections(const rsvd_ctx *ctx, rsvd_dtype dtype, int64_t l, int batch) {
  return l >= 16 && l <= corr_max_order(dtype == RSVD_F32) && batch <= ctx->cu_count &&
         jacobi_lds_bytes(dtype, l) + corr_lds_bytes(dtype, l) + 4096 <= ctx->lds_per_block;
}

hipError_t jacobi_launch(rsvd_ctx *ctx, hipStream_t s, rsvd_dtype dtype, int64_t l, const void *M,
                         int m_is_f64, const SigmaOut &sig, void *X, void *W, DevInfo *info, void *scratch,
                         size_t scratch_bytes, int batch, int64_t stride, int rows, const JacobiSlots *slots) {
  if (batch < 1 || batch > 65535) return hipErrorInvalidValue;
  if (l > jacobi_max_lds_order(ctx, dtype) || (batch == 1 && slots != nullptr && m_is_f64 && jacobi_prefers_blocks(dtype, l))) {
    if (batch != 1) {
      // the block path is not batched: fp64 orders up to 128 take the one-workgroup kernel with J in global memory
      // (the block path's scratch, which every problem of the batch has, is larger than one J)
      if (dtype != RSVD_F64 || l > jacobi_max_batched_order(ctx, dtype) || !m_is_f64 || scratch == nullptr ||
          scratch_bytes < jacobi_jglobal_bytes(l))
        return hipErrorNotSupported;
      const int ldm = jacobi_ldm((int)l, 16, 8);
      const size_t lds = align_up((size_t)l * ldm * 8 + (size_t)l * (8 + sizeof(int)), 16);
      const int nt = (int)align_up((size_t)((l + 1) / 2) * 16, 64);
      ProfScope ps(ctx, s, PK_JACOBI);
      if (jacobi_rows_padded((int)l, 16, 8) / 16 == 7)
        return launch_lds_jg<7>(s, nt, lds, M, (int)l, sig, X, W, info, batch, stride, rows, scratch);
      return launch_lds_jg<8>(s, nt, lds, M, (int)l, sig, X, W, info, batch, stride, rows, scratch);
    }
    // block path: needs the fp64 input (the triangular factor) and its scratch
    const size_t need = jacobi_scratch_bytes(ctx, dtype, l);
    if (l > jacobi_max_lds_order(ctx, dtype) && (need == 0 || scratch == nullptr || scratch_bytes < need || !m_is_f64))
      return hipErrorNotSupported;
    if (dtype == RSVD_F32)
      return jacobi_block_launch<float>(ctx, s, dtype, (int)l, (const double *)M, sig, (float *)X,
                                        (float *)W, info, (char *)scratch, rows, slots);
    return jacobi_block_launch<double>(ctx, s, dtype, (int)l, (const double *)M, sig, (double *)X,
                                       (double *)W, info, (char *)scratch, rows, slots);
  }
  // one G-lane group per column pair of a round, all pairs of a round at once
  const int npairs = (int)((l + 1) / 2);
  const int G = jacobi_group(dtype, l);
  int nt = (int)align_up((size_t)npairs * G, 64);
  if (nt > 64 * G) nt = 64 * G;
  const int g = jacobi_rows_padded((int)l, G, (int)dtype_size(dtype)) / G;          // rows per lane
  size_t lds = jacobi_lds_bytes(dtype, l);
  const bool corrections = lds_takes_corrections(ctx, dtype, l, batch);
  if (corrections) {
    lds += corr_lds_bytes(dtype, l);
    // Four wavefronts for each 16 rows: the products have work for nb * corr_strips(nb) of them, loads and stores for more, and every one
    // waits at the barriers of a sweep (fp32 l = 32, one sweep of equal values and all of a Gaussian factor, us: 4 wavefronts 18.6, 66.6; 8 17.2, 65.4; 16 17.7, 66.7).
    const int waves = 4 * (int)ceil_div(l, 16);
    nt = 64 * (waves < kCorrWaves ? waves : kCorrWaves);
  }
  ProfScope ps(ctx, s, PK_JACOBI);
  if (dtype == RSVD_F32) {
    if (m_is_f64) return launch_lds_g<float, double>(s, nt, G, g, lds, M, (int)l, sig, X, W, info, batch, stride, rows, corrections);
    return launch_lds_g<float, float>(s, nt, G, g, lds, M, (int)l, sig, X, W, info, batch, stride, rows, corrections);
  }
  return launch_lds_g<double, double>(s, nt, G, g, lds, M, (int)l, sig, X, W, info, batch, stride, rows, corrections);
}

}  // namespace rsvd
