// The r x r solve of every update through a Cholesky factorisation, on fp64 MFMA.
//
// The least-squares step needs (P_J^T P_J)^-1 (eqs. lsqA, lsqA_sto).  With G = P_J^T P_J
// symmetric positive definite, G = L L^T (Cholesky), and G^-1 = M^T M with M = L^-1.  The
// apply multiplies by -G^-1 as one matrix product, so that is what is formed here:
//
//   1. L by blocks of NB columns, left-looking: launch k has one workgroup per block row
//      i >= k.  Each computes the updated diagonal block A_kk - sum_{l<k} L_kl L_kl^T, factors
//      it (every workgroup of the launch does so, which removes any dependence between them),
//      forms D_k = L_kk^-1 and, for i > k, L_ik = (A_ik - sum_{l<k} L_il L_kl^T) D_k^T.
//   2. M = L^-1 by block columns (one workgroup each): M_jj = D_j and, for i > j,
//      M_ij = -D_i sum_{l=j}^{i-1} L_il M_lj.
//   3. -G^-1 = -M^T M by 64 x 64 tiles: tile (a, b) = -sum_{l >= max(a, b)} M_la^T M_lb.
//
// The launches take a batch of matrices (blockIdx.y), each with its own work area and step id.
// A matrix of one block (r_p <= 64) takes a single launch with its Gram matrix (solve_small_kernel
// below).  A pivot that is not positive (or not finite) flags that step as not positive definite;
// its apply and the later ones then write nothing.  Blocks of NB x NB doubles are staged in LDS
// with row stride NB + 1; fp64 MFMA v_mfma_f64_16x16x4f64: srcA lane l = A[l % 16][l / 16], srcB
// lane l = B[l / 16][l % 16], accumulator register v of lane l = D[4 v + l / 16][l % 16].

#include <algorithm>

#include "sparse_terms.h"

namespace nmd {

typedef double dx4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kThreads = 1024;

// Work area of matrix b: L, M = L^-1, -G^-1 (rp x rp each) and the diagonal blocks D_k.
struct Work {
  double *L, *M, *Gneg, *D;
  __host__ __device__ Work(double* base, int64_t per, int b, int rp) {
    double* w = base + per * b;
    L = w;
    M = w + (int64_t)rp * rp;
    Gneg = w + 2 * (int64_t)rp * rp;
    D = w + 3 * (int64_t)rp * rp;
  }
};

// Copies the NB x NB block at (bi, bj) of a row-major matrix with leading dimension ld into LDS.
template <int NB>
__device__ __forceinline__ void stage(double* dst, const double* __restrict__ src, int ld, int bi,
                                      int bj) {
  constexpr int LS = NB + 1;
  for (int e = threadIdx.x; e < NB * NB; e += kThreads) {
    const int r = e / NB, c = e - r * NB;
    dst[r * LS + c] = src[(int64_t)(bi * NB + r) * ld + bj * NB + c];
  }
}

// acc += A B^T for two NB x NB blocks in LDS: (A B^T)[r][c] = sum_m A[r][m] B[c][m]; wave w
// owns the 16 x 16 output sub-tile (w / (NB / 16), w % (NB / 16)).
template <int NB>
__device__ __forceinline__ void mma_abt(dx4& acc, const double* A, const double* B, int ri,
                                        int ci, int q, int l16) {
  constexpr int LS = NB + 1;
#pragma unroll 4
  for (int m0 = 0; m0 < NB; m0 += 4) {
    const double a = A[(16 * ri + l16) * LS + m0 + q];
    const double b = B[(16 * ci + l16) * LS + m0 + q];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
  }
}

// acc += A^T B: (A^T B)[r][c] = sum_m A[m][r] B[m][c].
template <int NB>
__device__ __forceinline__ void mma_atb(dx4& acc, const double* A, const double* B, int ri,
                                        int ci, int q, int l16) {
  constexpr int LS = NB + 1;
#pragma unroll 4
  for (int m0 = 0; m0 < NB; m0 += 4) {
    const double a = A[(m0 + q) * LS + 16 * ri + l16];
    const double b = B[(m0 + q) * LS + 16 * ci + l16];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
  }
}

// acc += A B: (A B)[r][c] = sum_m A[r][m] B[m][c].
template <int NB>
__device__ __forceinline__ void mma_ab(dx4& acc, const double* A, const double* B, int ri, int ci,
                                       int q, int l16) {
  constexpr int LS = NB + 1;
#pragma unroll 4
  for (int m0 = 0; m0 < NB; m0 += 4) {
    const double a = A[(16 * ri + l16) * LS + m0 + q];
    const double b = B[(m0 + q) * LS + 16 * ci + l16];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
  }
}

// Writes s * acc (the wave's sub-tile) into an LDS block.
template <int NB>
__device__ __forceinline__ void put_tile(double* dst, const dx4& acc, double s, int ri, int ci,
                                         int q, int l16) {
  constexpr int LS = NB + 1;
#pragma unroll
  for (int v = 0; v < 4; ++v) dst[(16 * ri + 4 * v + q) * LS + 16 * ci + l16] = s * acc[v];
}

// 1 / sqrt(x) for normal x > 0 to about an ulp: the hardware estimate (2^-14 or better)
// refined by Newton steps, each of which doubles its correct bits.  Pivots are sums of products of
// fp32 numbers, far inside the range of normal doubles.
__device__ __forceinline__ double recip_sqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int k = 0; k < 3; ++k) y = fma(y * 0.5, fma(-x * y, y, 1.0), y);
  return y;
}

__device__ __forceinline__ double lane_value(double x, int lane) {
  const long long b = __builtin_bit_cast(long long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// W with W^T W = P^-1 for a symmetric positive definite 4 x 4 P (p: its lower triangle by rows),
// W = L^-1 of its Cholesky factor, lower triangular by rows.  False if a pivot was not positive
// (or not finite).
__device__ __forceinline__ bool inv_chol4(const double (&p)[10], double (&w)[10]) {
  double l[10];
  bool ok = true;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int jj = j * (j + 1) / 2;
    double d = p[jj + j];
#pragma unroll
    for (int m = 0; m < j; ++m) d = fma(-l[jj + m], l[jj + m], d);
    const bool good = d > 0.0 && d < __builtin_huge_val();
    ok = ok && good;
    const double s = recip_sqrt(good ? d : 1.0);
#pragma unroll
    for (int i = j + 1; i < 4; ++i) {
      const int ii = i * (i + 1) / 2;
      double x = p[ii + j];
#pragma unroll
      for (int m = 0; m < j; ++m) x = fma(-l[ii + m], l[jj + m], x);
      l[ii + j] = x * s;
    }
    // row j of W: w_jj = s, w_ji = -s sum_{m=i}^{j-1} l_jm w_mi
    w[jj + j] = s;
#pragma unroll
    for (int i = 0; i < j; ++i) {
      double x = 0.0;
#pragma unroll
      for (int m = i; m < j; ++m) x = fma(l[jj + m], w[m * (m + 1) / 2 + i], x);
      w[jj + i] = -s * x;
    }
  }
  return ok;
}

// D with D^T D = A^-1 for the symmetric 16 x 16 block at A (row stride LS), lower triangular (the
// inverse of its Cholesky factor), by one wave, into `inv`.  Elimination of [A | E], E = I at the
// start, four rows at a time, in the accumulator layout (register v of lane (q, l16): row 4 v + q,
// column l16).  Step J takes the block row R = rows 4 J .. 4 J + 3, which is register J as it
// stands, and its pivot block P = W^-1 W^-T: S = W R is one matrix instruction whose result is
// rows 4 J .. of L^T (register 0: row k in lanes q = k), and A -= S^T S, E -= S^T (W E_J), with S
// as both operands as it stands (A operand lane (l16, q): column l16 of row q; B the same).
// W E_J are rows 4 J .. of D.  So each step is four pivots in scalar arithmetic and four matrix
// instructions; a step per column (a pivot and two instructions) took 500 cycles a column.
// Returns false if a pivot was not positive (or not finite).
template <int LS>
__device__ __forceinline__ bool factor16(const double* A, double* inv, int q, int l16) {
  dx4 a, e;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    a[v] = A[(4 * v + q) * LS + l16];
    e[v] = 4 * v + q == l16 ? 1.0 : 0.0;
  }
  bool ok = true;
#pragma unroll
  for (int J = 0; J < 4; ++J) {
    double p[10], w[10];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int k = 0; k <= i; ++k) p[i * (i + 1) / 2 + k] = lane_value(a[J], 16 * k + 4 * J + i);
    ok = inv_chol4(p, w) && ok;
    // A operand of the products with W: lane (l16 = i, q = k) holds W[i][k], zero outside
    double wa = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int k = 0; k <= i; ++k)
        if (l16 == i && q == k) wa = w[i * (i + 1) / 2 + k];
    const dx4 zero = {0.0, 0.0, 0.0, 0.0};
    const dx4 sr = __builtin_amdgcn_mfma_f64_16x16x4f64(wa, a[J], zero, 0, 0, 0);
    const dx4 se = __builtin_amdgcn_mfma_f64_16x16x4f64(wa, e[J], zero, 0, 0, 0);
    inv[(4 * J + q) * LS + l16] = se[0];
    if (J < 3) {
      // only rows past the block row: the others are done
      const double f = l16 > 4 * J + 3 ? -sr[0] : 0.0;
      a = __builtin_amdgcn_mfma_f64_16x16x4f64(f, sr[0], a, 0, 0, 0);
      e = __builtin_amdgcn_mfma_f64_16x16x4f64(f, se[0], e, 0, 0, 0);
    }
  }
  return ok;
}

// acc += A B^T, A B of 16 x 16 blocks at A and B (row stride LS).
template <int LS>
__device__ __forceinline__ void mma16_abt(dx4& acc, const double* A, const double* B, int q,
                                          int l16) {
#pragma unroll
  for (int m0 = 0; m0 < 16; m0 += 4)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(A[l16 * LS + m0 + q], B[l16 * LS + m0 + q], acc, 0, 0, 0);
}
template <int LS>
__device__ __forceinline__ void mma16_ab(dx4& acc, const double* A, const double* B, int q,
                                         int l16) {
#pragma unroll
  for (int m0 = 0; m0 < 16; m0 += 4)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(A[l16 * LS + m0 + q], B[(m0 + q) * LS + l16], acc, 0, 0, 0);
}

// D = L^-1 (lower triangular, zeros above) of the Cholesky factor of the symmetric NB x NB block A
// in LDS, into `inv`, by 16 x 16 sub-blocks: for each block column one wave inverts the factor of
// the diagonal sub-block, then L_ik = A_ik D_k^T and A_ij -= L_ik L_jk^T on a wave per sub-block; then the
// sub-diagonals of the inverse, M_ij = -D_i sum_{l=j}^{i-1} L_il M_lj.  Three barriers per block
// column and one per sub-diagonal instead of one per column, whose 64 rounds of barrier, LDS
// reads and reciprocal were nearly all of the solve's time.  A's off-diagonal sub-blocks below the
// diagonal become those of L.  Returns false, in every thread, if a pivot was not positive (or
// not finite).
template <int NB>
__device__ bool factor_block(double* A, double* inv) {
  constexpr int LS = NB + 1;
  constexpr int NT = NB / 16;
  __shared__ int bad;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int q = lane >> 4, l16 = lane & 15;
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();
  auto at = [](double* m, int i, int j) { return m + 16 * i * LS + 16 * j; };
#pragma unroll 1
  for (int k = 0; k < NT; ++k) {
    if (wave == 0) {
      const bool ok = factor16<LS>(at(A, k, k), at(inv, k, k), q, l16);
      if (!ok && lane == 0) bad = 1;
    }
    __syncthreads();
    if (wave > k && wave < NT) {  // L_ik, i = wave
      double* t = at(A, wave, k);
      dx4 o = {0.0, 0.0, 0.0, 0.0};
      mma16_abt<LS>(o, t, at(inv, k, k), q, l16);
#pragma unroll
      for (int v = 0; v < 4; ++v) t[(4 * v + q) * LS + l16] = o[v];
    }
    __syncthreads();
    // A_ij -= L_ik L_jk^T for k < j <= i: wave = 4 i + j
    const int i = wave >> 2, j = wave & 3;
    if (i < NT && j > k && j <= i) {
      double* t = at(A, i, j);
      dx4 o = {0.0, 0.0, 0.0, 0.0};
      mma16_abt<LS>(o, at(A, i, k), at(A, j, k), q, l16);
#pragma unroll
      for (int v = 0; v < 4; ++v) t[(4 * v + q) * LS + l16] -= o[v];
    }
    __syncthreads();
  }
  // zeros above the diagonal sub-blocks of the inverse, then its sub-diagonals
  for (int e = threadIdx.x; e < NB * NB; e += kThreads) {
    const int r = e / NB, c = e - r * NB;
    if (c / 16 > r / 16) inv[r * LS + c] = 0.0;
  }
#pragma unroll 1
  for (int d = 1; d < NT; ++d) {
    const int i = wave + d, j = wave;
    if (i < NT) {
      dx4 t = {0.0, 0.0, 0.0, 0.0};
      for (int l = j; l < i; ++l) mma16_ab<LS>(t, at(A, i, l), at(inv, l, j), q, l16);
      dx4 o = {0.0, 0.0, 0.0, 0.0};
      // register s of t is row 4 s + q of the product: the B operand of k-step s as it stands
      const double* di = at(inv, i, i);
#pragma unroll
      for (int m = 0; m < 4; ++m)
        o = __builtin_amdgcn_mfma_f64_16x16x4f64(di[l16 * LS + 4 * m + q], t[m], o, 0, 0, 0);
      double* dst = at(inv, i, j);
#pragma unroll
      for (int v = 0; v < 4; ++v) dst[(4 * v + q) * LS + l16] = -o[v];
    }
    __syncthreads();
  }
  const bool ok = bad == 0;
  __syncthreads();
  return ok;
}

}  // namespace

// Launch k of step 1: block row i = k + blockIdx.x of matrix blockIdx.y.
template <int NB>
__global__ __launch_bounds__(kThreads) void chol_col_kernel(const double* __restrict__ Gall,
                                                            double* __restrict__ work,
                                                            int64_t per, int rp, int k,
                                                            int* status, SolveBatch sb) {
  constexpr int LS = NB + 1;
  constexpr int NT = NB / 16;  // sub-tiles per dimension
  __shared__ double sA[NB * LS], sB[NB * LS], s1[NB * LS], s2[NB * LS];
  const Work wk(work, per, blockIdx.y, rp);
  const double* __restrict__ G = Gall + (int64_t)blockIdx.y * rp * rp;
  double* __restrict__ L = wk.L;
  double* __restrict__ D = wk.D;
  const int i = k + blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int q = lane >> 4, l16 = lane & 15;
  const bool mw = wave < NT * NT;  // waves with an output sub-tile
  const int ri = wave / NT, ci = wave % NT;
  dx4 akk = {0.0, 0.0, 0.0, 0.0}, aik = {0.0, 0.0, 0.0, 0.0};
  for (int l = 0; l < k; ++l) {
    __syncthreads();
    stage<NB>(s1, L, rp, k, l);
    if (i != k) stage<NB>(s2, L, rp, i, l);
    __syncthreads();
    if (mw) {
      mma_abt<NB>(akk, s1, s1, ri, ci, q, l16);
      if (i != k) mma_abt<NB>(aik, s2, s1, ri, ci, q, l16);
    }
  }
  stage<NB>(sA, G, rp, k, k);
  if (i != k) stage<NB>(sB, G, rp, i, k);
  __syncthreads();
  if (mw) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int o = (16 * ri + 4 * v + q) * LS + 16 * ci + l16;
      sA[o] -= akk[v];
      if (i != k) sB[o] -= aik[v];
    }
  }
  const bool ok = factor_block<NB>(sA, s1);  // s1 = D_k = L_kk^-1
  if (!ok && blockIdx.x == 0 && threadIdx.x == 0)
    flag_status(status, STATUS_NOTPD, sb.step_id[blockIdx.y]);
  if (i == k) {
    for (int e = threadIdx.x; e < NB * NB; e += kThreads) {
      const int r = e / NB, c = e - r * NB;
      D[(int64_t)k * NB * NB + e] = s1[r * LS + c];
    }
    return;
  }
  // L_ik = A_ik D_k^T
  dx4 o = {0.0, 0.0, 0.0, 0.0};
  if (mw) mma_abt<NB>(o, sB, s1, ri, ci, q, l16);
  if (mw) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
      L[(int64_t)(i * NB + 16 * ri + 4 * v + q) * rp + k * NB + 16 * ci + l16] = o[v];
  }
}

// Step 2 for block column j of M = L^-1 (rows i >= j): M_jj = D_j and, for i > j,
// M_ij = -D_i sum_{l=j}^{i-1} L_il M_lj.  Four NB x NB LDS blocks; ends with the LDS free once
// the caller synchronises.
template <int NB>
__device__ void trinv_column(const double* __restrict__ L, const double* __restrict__ D,
                             double* __restrict__ Mb, int rp, int j, double* sL, double* sM,
                             double* sT, double* sD) {
  constexpr int LS = NB + 1;
  constexpr int NT = NB / 16;
  const int nb = rp / NB;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int q = lane >> 4, l16 = lane & 15;
  const bool mw = wave < NT * NT;
  const int ri = wave / NT, ci = wave % NT;
  for (int e = threadIdx.x; e < NB * NB; e += kThreads) {
    const int r = e / NB, c = e - r * NB;
    Mb[(int64_t)(j * NB + r) * rp + j * NB + c] = D[(int64_t)j * NB * NB + e];
  }
  for (int i = j + 1; i < nb; ++i) {
    dx4 t = {0.0, 0.0, 0.0, 0.0};
    for (int l = j; l < i; ++l) {
      __syncthreads();  // Mb writes of the previous block row are visible; LDS is free
      stage<NB>(sL, L, rp, i, l);
      stage<NB>(sM, Mb, rp, l, j);
      __syncthreads();
      if (mw) mma_ab<NB>(t, sL, sM, ri, ci, q, l16);
    }
    __syncthreads();
    if (mw) put_tile<NB>(sT, t, 1.0, ri, ci, q, l16);
    for (int e = threadIdx.x; e < NB * NB; e += kThreads) {
      const int r = e / NB, c = e - r * NB;
      sD[r * LS + c] = D[(int64_t)i * NB * NB + e];
    }
    __syncthreads();
    dx4 o = {0.0, 0.0, 0.0, 0.0};
    if (mw) mma_ab<NB>(o, sD, sT, ri, ci, q, l16);
    if (mw) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        Mb[(int64_t)(i * NB + 16 * ri + 4 * v + q) * rp + j * NB + 16 * ci + l16] = -o[v];
    }
  }
}

// Step 2: block column j = blockIdx.x of matrix blockIdx.y.
template <int NB>
__global__ __launch_bounds__(kThreads) void chol_trinv_kernel(double* __restrict__ work,
                                                              int64_t per, int rp) {
  constexpr int LS = NB + 1;
  __shared__ double sL[NB * LS], sM[NB * LS], sT[NB * LS], sD[NB * LS];
  const Work wk(work, per, blockIdx.y, rp);
  trinv_column<NB>(wk.L, wk.D, wk.M, rp, blockIdx.x, sL, sM, sT, sD);
}

// Step 3 for tile (a, b), a <= b, of -G^-1 = -M^T M: -sum_{l >= b} M_la^T M_lb, written to
// both (a, b) and (b, a).  Two NB x NB LDS blocks.
template <int NB>
__device__ void gram_tile(const double* __restrict__ Mb, double* __restrict__ Gneg, int rp, int a,
                          int b, double* s1, double* s2) {
  constexpr int NT = NB / 16;
  const int nb = rp / NB;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int q = lane >> 4, l16 = lane & 15;
  const bool mw = wave < NT * NT;
  const int ri = wave / NT, ci = wave % NT;
  dx4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int l = b; l < nb; ++l) {
    __syncthreads();
    stage<NB>(s1, Mb, rp, l, a);
    stage<NB>(s2, Mb, rp, l, b);
    __syncthreads();
    if (mw) mma_atb<NB>(acc, s1, s2, ri, ci, q, l16);
  }
  if (mw) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * ri + 4 * v + q, c = 16 * ci + l16;
      Gneg[(int64_t)(a * NB + r) * rp + b * NB + c] = -acc[v];
      if (a != b) Gneg[(int64_t)(b * NB + c) * rp + a * NB + r] = -acc[v];
    }
  }
}

// Pair index p -> tile (a, b) with a <= b, in the order (0,0), (0,1), ..., (1,1), ...
__device__ __forceinline__ void tile_pair(int p, int nb, int& a, int& b) {
  a = 0;
  while (p >= nb - a) {
    p -= nb - a;
    ++a;
  }
  b = a + p;
}

// Step 3: tile pair blockIdx.x of matrix blockIdx.y.
template <int NB>
__global__ __launch_bounds__(kThreads) void chol_gram_kernel(double* __restrict__ work,
                                                             int64_t per, int rp,
                                                             const int* status, SolveBatch sb) {
  constexpr int LS = NB + 1;
  __shared__ double s1[NB * LS], s2[NB * LS];
  const Work wk(work, per, blockIdx.y, rp);
  int a, b;
  tile_pair(blockIdx.x, rp / NB, a, b);
  if (step_blocked(status, sb.step_id[blockIdx.y])) return;  // its apply writes nothing
  gram_tile<NB>(wk.M, wk.Gneg, rp, a, b, s1, s2);
}

// The whole solve of a matrix of one block, T = r_p <= 64, from the panel: workgroup (c, b) forms
// chunk c of the Gram matrix of batch entry b, and the last one to finish sums the chunks (in
// order), factors the sum and writes -G^-1 = -D^T D.  At these ranks three launches (Gram,
// reduction, factorisation) took 60 us a step for 25 us of work, most of it waiting for each
// other's launch and for the sum of two or three chunks.
//
// The operands come straight from memory: wave w takes the 16 x 16 tile w % NS of the upper
// triangle and every KSP-th group of four panel rows (16 waves, NS tiles), so no wave waits for
// another before the chunk ends; at T = 64 ten waves share four fp64 matrix units, which bounds
// it (64 rows 1.3 us).
constexpr int kSmallChunks = 16;
constexpr int small_tiles(int T) { return (T / 16) * (T / 16 + 1) / 2; }

template <int T>
__device__ __forceinline__ void solve_small(int c, int b, const float* __restrict__ P,
                                            const SolveBatch& sb, int r, double* __restrict__ part,
                                            int nchunks, int* __restrict__ done,
                                            double* __restrict__ Gneg_all, int* status) {
  constexpr int NT = T / 16, LS = T + 1, NS = small_tiles(T), KSP = 16 / NS;
  constexpr int NE = NS * 256;                          // elements of a chunk's partial
  constexpr int PT = (NE + kThreads - 1) / kThreads;    // of them per thread
  constexpr int RED = KSP * NE, MAT = 2 * T * LS;
  __shared__ double buf[RED > MAT ? RED : MAT];
  __shared__ int last;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int q = lane >> 4, l16 = lane & 15;
  const int64_t k0 = (int64_t)c * sb.blk[b] / nchunks, k1 = (int64_t)(c + 1) * sb.blk[b] / nchunks;
  // tile t of the upper triangle: rows 16 ti .., columns 16 tj ..
  auto tile_of = [](int t, int& ti, int& tj) {
    ti = 0;
    while (t >= NT - ti) {
      t -= NT - ti;
      ++ti;
    }
    tj = ti + t;
  };
  if (wave < NS * KSP) {
    const int t = wave % NS, kp = wave / NS;
    int ti, tj;
    tile_of(t, ti, tj);
    constexpr int U = 8;
    dx4 acc = {0.0, 0.0, 0.0, 0.0};
    const float* base = P + sb.j0[b] * T;
    float an[U], bn[U];  // the next round's rows, in flight during this round's products
    auto fetch = [&](int64_t k) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t row = k + 4 * KSP * u + q;
        const float* src = base + (row < k1 ? row : k0) * T;  // a row past the end counts zero
        an[u] = src[16 * ti + l16];
        bn[u] = src[16 * tj + l16];
        if (row >= k1) an[u] = bn[u] = 0.f;
      }
    };
    const int64_t first = k0 + 4 * kp;
    if (first < k1) fetch(first);
    for (int64_t k = first; k < k1; k += 4 * KSP * U) {
      float av[U], bv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        av[u] = an[u];
        bv[u] = bn[u];
      }
      if (k + 4 * KSP * U < k1) fetch(k + 4 * KSP * U);
#pragma unroll
      for (int u = 0; u < U; ++u)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)av[u], (double)bv[u], acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) buf[(kp * NS + t) * 256 + (4 * v + q) * 16 + l16] = acc[v];
  }
  __syncthreads();
  double g[PT];
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    const int e = tid + kThreads * i;
    g[i] = 0.0;
    if (e < NE) {
#pragma unroll
      for (int kp = 0; kp < KSP; ++kp) g[i] += buf[kp * NE + e];
    }
  }
  if (nchunks > 1) {
    double* mine = part + (int64_t)(b * nchunks + c) * NE;
#pragma unroll
    for (int i = 0; i < PT; ++i)
      if (tid + kThreads * i < NE) mine[tid + kThreads * i] = g[i];
    // Every wave waits until its stores have reached the L2: the barrier does not (it is enough for
    // the waves of one CU, which share a vector cache), and the write-back below waits for its own
    // wave's only, while the reader may run on another XCD, behind another L2.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // one thread releases the workgroup's partial and acquires the others' (every wave doing so
    // took 7 us); the count returns to zero for the next launch
    if (tid == 0)
      last = __hip_atomic_fetch_add(&done[b], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) ==
             nchunks - 1;
    __syncthreads();
    if (!last) return;
    if (tid == 0) done[b] = 0;
    const double* all = part + (int64_t)b * nchunks * NE;
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int e = tid + kThreads * i;
      g[i] = 0.0;
      if (e < NE) {
        // all partials requested together, added in order
        double x[kSmallChunks];
#pragma unroll
        for (int k = 0; k < kSmallChunks; ++k)
          x[k] = all[(int64_t)(k < nchunks ? k : nchunks - 1) * NE + e];
#pragma unroll
        for (int k = 0; k < kSmallChunks; ++k) g[i] += k < nchunks ? x[k] : 0.0;
      }
    }
  }
  __syncthreads();  // the tiles in buf have been read
  double* A = buf;
  double* D = buf + T * LS;
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    const int e = tid + kThreads * i;
    if (e >= NE) continue;
    int ti, tj;
    tile_of(e / 256, ti, tj);
    const int row = 16 * ti + (e & 255) / 16, col = 16 * tj + (e & 15);
    const double x = row < r && col < r ? g[i] : (row == col ? 1.0 : 0.0);
    A[row * LS + col] = x;
    A[col * LS + row] = x;
  }
  if (!factor_block<T>(A, D)) {
    if (tid == 0) flag_status(status, STATUS_NOTPD, sb.step_id[b]);
    return;
  }
  double* Gneg = Gneg_all + (int64_t)b * T * T;
  if (wave < NT * NT) {
    const int ri = wave / NT, ci = wave % NT;
    dx4 acc = {0.0, 0.0, 0.0, 0.0};
    mma_atb<T>(acc, D, D, ri, ci, q, l16);
#pragma unroll
    for (int v = 0; v < 4; ++v) Gneg[(16 * ri + 4 * v + q) * T + 16 * ci + l16] = -acc[v];
  }
}

template <int T>
__global__ __launch_bounds__(kThreads) void solve_small_kernel(const float* __restrict__ P,
                                                               SolveBatch sb, int r,
                                                               double* __restrict__ part,
                                                               int nchunks, int* __restrict__ done,
                                                               double* __restrict__ Gneg_all,
                                                               int* status) {
  solve_small<T>(blockIdx.x, blockIdx.y, P, sb, r, part, nchunks, done, Gneg_all, status);
}

// The same with a small step's sparse correction in the launch's other workgroups: neither needs
// the other's result, and each alone leaves most of the chip idle (5003 x 2999, r = 40: 18 and
// 17 us one after the other, 1.37 ms a fit; in one launch 1.06 ms).  The first sb.n nchunks workgroups solve; of the others `threads`
// threads take the correction's items, or rows where it walks rows (rowptr != nullptr).
template <int T>
__global__ __launch_bounds__(kThreads) void solve_sparse_kernel(
    const float* __restrict__ P, SolveBatch sb, int r, double* __restrict__ part, int nchunks,
    int* __restrict__ done, double* __restrict__ Gneg_all, int* status, SparseWork w, int threads) {
  const int nsolve = sb.n * nchunks;
  if ((int)blockIdx.x < nsolve) {
    solve_small<T>(blockIdx.x % nchunks, blockIdx.x / nchunks, P, sb, r, part, nchunks, done, Gneg_all,
                   status);
    return;
  }
  if ((int)threadIdx.x >= threads) return;
  constexpr int E = T / 16;
  const int64_t thread = (int64_t)(blockIdx.x - nsolve) * threads + threadIdx.x;
  if (w.rowptr)
    sparse_row<16, E, 2 * kDepth, contig(E)>(thread >> 6, w.rowptr, w.nblk, w.rows, w.idx, w.val, w.X,
                                             w.P, w.Y, 1);
  else
    sparse_item<16, E, kDepth, contig(E)>(thread, w.items, w.nitems, w.idx, w.val, w.X, w.P, w.Y,
                                          w.scratch, 1);
}

int solve_small_chunks(int rp, int64_t blk, int n) {
  // panel rows per chunk: what the waves request in one round (two at r_p = 64), or so many that
  // sixteen chunks cover the panel (the last workgroup reads them all)
  const int64_t rows = rp == 16 ? 512 : (rp == 32 ? 160 : 64);
  const int64_t most = std::min<int64_t>(kSmallChunks, kGramChunks / n);
  return (int)std::max<int64_t>(1, std::min<int64_t>((blk + rows - 1) / rows, most));
}

hipError_t launch_solve_small(const float* P, const SolveBatch& sb, int r, int rp, double* part,
                              int nchunks, int* done, double* work, int* status, double** result,
                              hipStream_t st) {
  if (sb.n < 1 || sb.n > kSolveBatch || nchunks < 1 || nchunks > kSmallChunks ||
      nchunks * sb.n > kGramChunks)
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)nchunks, (unsigned)sb.n);
#define SMALL(T)                                                                              \
  hipLaunchKernelGGL((solve_small_kernel<T>), grid, dim3(kThreads), 0, st, P, sb, r, part,      \
                     nchunks, done, work, status)
  switch (rp) {
    case 16: SMALL(16); break;
    case 32: SMALL(32); break;
    case 48: SMALL(48); break;
    case 64: SMALL(64); break;
    default: return hipErrorInvalidValue;
  }
#undef SMALL
  for (int b = 0; b < sb.n; ++b) result[b] = work + (int64_t)b * rp * rp;
  return hipGetLastError();
}

hipError_t launch_solve_sparse(const float* P, const SolveBatch& sb, int r, int rp, double* part,
                               int nchunks, int* done, double* work, int* status,
                               const SparseWork& w, hipStream_t st) {
  if (sb.n < 1 || sb.n > kSolveBatch || nchunks < 1 || nchunks > kSmallChunks ||
      nchunks * sb.n > kGramChunks)
    return hipErrorInvalidValue;
  const int64_t need = w.rowptr ? 64 * w.rows : 16 * w.nitems;
  // 256 threads per workgroup while that leaves a CU each (63 workgroups of 16 rows leave three
  // quarters of the chip idle), else all of them
  const int threads = need <= 256 * 256 ? 256 : kThreads;
  const int64_t total = (int64_t)sb.n * nchunks + (need + threads - 1) / threads;
  if (total > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)total);
#define SMALL(T)                                                                              \
  hipLaunchKernelGGL((solve_sparse_kernel<T>), grid, dim3(kThreads), 0, st, P, sb, r, part,     \
                     nchunks, done, work, status, w, threads)
  switch (rp) {
    case 16: SMALL(16); break;
    case 32: SMALL(32); break;
    case 48: SMALL(48); break;
    case 64: SMALL(64); break;
    default: return hipErrorInvalidValue;
  }
#undef SMALL
  return hipGetLastError();
}

constexpr int kBlock = 64;  // columns of a block, r_p >= 128 (below, launch_solve_small)

int64_t chol_work_doubles(int rp) { return 3 * (int64_t)rp * rp + (int64_t)rp * kBlock; }

hipError_t launch_chol_inverse(const double* G, double* work, int rp, int* status,
                               const SolveBatch& sb, double** result, hipStream_t st) {
  if (sb.n < 1 || sb.n > kSolveBatch || rp % kBlock) return hipErrorInvalidValue;
  const int nb = rp / kBlock;
  const int64_t per = chol_work_doubles(rp);
  const unsigned nm = (unsigned)sb.n;
  for (int k = 0; k < nb; ++k) {
    hipLaunchKernelGGL((chol_col_kernel<kBlock>), dim3(nb - k, nm), dim3(kThreads), 0, st, G, work, per,
                       rp, k, status, sb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((chol_trinv_kernel<kBlock>), dim3(nb, nm), dim3(kThreads), 0, st, work, per, rp);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((chol_gram_kernel<kBlock>), dim3(nb * (nb + 1) / 2, nm), dim3(kThreads), 0, st, work,
                     per, rp, status, sb);
  for (int b = 0; b < sb.n; ++b) result[b] = Work(work, per, b, rp).Gneg;
  return hipGetLastError();
}

}  // namespace nmd
