// The objective and the reconstruction measures (sums q0 .. q4 of objective.hip) with L on bf16
// MFMA of three-term splits (split_wide.h), for r_p a multiple of 64.
//
// The producers are the contraction's; a consumer takes the terms of its 32 x 32 tiles of L from
// LDS, one block behind them.  Each lane owns one row and four of every eight columns (at r_p >
// 128, where two consumers share a tile, of every other sixteen), and walks the row's nonzeros in
// step with the blocks: the walk keeps two entries ahead in registers, so that taking one does not
// wait for the next.  Every term is taken once from one L, as in objective.hip: an entry takes
// its own terms and zeroes its L before the branch-free pass that adds max(0, L)^2 for the others.
//
// What bounds it: the bf16 matrix rate, as the contraction without entries.  139255 x 139255, r = 256
// with 0.09% nonzeros: 82 -> 53 ms a call (fp32 MFMA before); the sums agree with the fp32 kernel's to
// its rounding, and their mean error is zero (two-term f16 splits, which drop the product of the low
// halves: -6e-9 of L).
//
// A workgroup that met a value outside the splits' range reports NaN, and objective.hip's kernel runs
// behind this one where the sum is NaN.

#include <climits>

#include "split_wide.h"

namespace nmd {
namespace sw {

struct Walk {
  int64_t ptr, end;
  int c0, c1;    // the next two entries' columns (INT_MAX: none)
  float v0, v1;  // and values
};

__device__ __forceinline__ void walk_next(Walk& w, const int32_t* __restrict__ idx,
                                          const float* __restrict__ val) {
  w.c0 = w.c1;
  w.v0 = w.v1;
  ++w.ptr;
  w.c1 = INT_MAX;
  if (w.ptr + 1 < w.end) {
    w.c1 = idx[w.ptr + 1];
    w.v1 = val[w.ptr + 1];
  }
}

// q[0] is q0 (or, without METRICS, q0 + q1), q[1] .. q[4] as in objective.hip.
template <int RP, bool METRICS>
__device__ __forceinline__ void tile_terms(double (&q)[5], Walk& w, const float* zt, int j0, int lo,
                                           int hi, int rg, int cp, int lane,
                                           const int32_t* __restrict__ idx,
                                           const float* __restrict__ val) {
  using C = Cfg<RP>;
  constexpr int NU = 4 / C::KS;  // groups of four registers this consumer takes
  const int h = lane >> 5;
  const float* src = zt + rg * C::KS * C::ZT + 4 * lane + 256 * NU * cp;
  const int jl = j0 + 8 * NU * cp + 4 * h;  // the lane's first column; group u: + 8 u
  float z[4 * NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    float4 a = *reinterpret_cast<const float4*>(src + 256 * u);
    if constexpr (C::KS == 2) {
      const float4 b = *reinterpret_cast<const float4*>(src + C::ZT + 256 * u);
      a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
    }
    z[4 * u] = a.x; z[4 * u + 1] = a.y; z[4 * u + 2] = a.z; z[4 * u + 3] = a.w;
  }
  if (j0 < lo || j0 + 32 > hi) {  // columns of the neighbouring ranges
#pragma unroll
    for (int v = 0; v < 4 * NU; ++v) {
      const int j = jl + 8 * (v >> 2) + (v & 3);
      if (j < lo || j >= hi) z[v] = 0.f;
    }
  }
  const int jend = j0 + 32 < hi ? j0 + 32 : hi;
  while (w.c0 < jend) {
    const int off = w.c0 - jl;
    if (off >= 0 && off < 8 * NU && (off & 7) < 4) {
      const int v = 4 * (off >> 3) + (off & 3);
      float lf = 0.f;
#pragma unroll
      for (int k = 0; k < 4 * NU; ++k)
        if (k == v) {
          lf = z[k];
          z[k] = 0.f;
        }
      const double sd = (double)w.v0;
      const double d = sd - (double)lf;
      if constexpr (METRICS) {
        const double p = (double)fmaxf(lf, 0.f);
        const double e = sd - p;
        q[1] += d * d;
        q[2] += e * e;
        q[3] += fmin(sd, p);
        q[4] += fmax(sd, p);
      } else {
        q[0] += d * d;
      }
    }
    walk_next(w, idx, val);
  }
  double s0 = 0.0, s1 = 0.0, t0 = 0.0, t1 = 0.0;
#pragma unroll
  for (int v = 0; v < 4 * NU; v += 2) {
    const double a = (double)fmaxf(z[v], 0.f), b = (double)fmaxf(z[v + 1], 0.f);
    s0 = fma(a, a, s0);
    s1 = fma(b, b, s1);
    if constexpr (METRICS) {
      t0 += a;
      t1 += b;
    }
  }
  q[0] += s0 + s1;
  if constexpr (METRICS) q[4] += t0 + t1;
}

// Workgroups over (row tile, column block, sub-split); partial[k * gridDim.x + workgroup] = its
// share of sum k.  The split panel covers all n columns in 32-column blocks from 0; a unit takes
// the blocks its columns touch and masks the others' columns.  Sub-splits start at whole blocks, so
// only the ends of a column block are taken twice (cut anywhere, sixteen ranges of 256 columns took
// three times the blocks).
template <int RP, bool METRICS>
__global__ __launch_bounds__(512, 2 * Cfg<RP>::WGS) void objective_split_kernel(
    const float* __restrict__ X, int64_t rows, const float* __restrict__ split,
    const int* __restrict__ bad_blocks, const int64_t* __restrict__ cbounds, int nsub,
    const int64_t* __restrict__ rowptr, const int32_t* __restrict__ idx,
    const float* __restrict__ val, int64_t row_tiles, double* __restrict__ partial) {
  using C = Cfg<RP>;
  constexpr int NQ = METRICS ? 5 : 1;
  __shared__ __attribute__((aligned(16))) float smem[C::LDS];
  __shared__ int bad;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  const int64_t logical = xcd_logical(blockIdx.x, (int64_t)gridDim.x);
  const int64_t unit = logical / row_tiles;
  const int64_t rt = logical - unit * row_tiles;
  const int b = (int)(unit / nsub), s = (int)(unit - (int64_t)b * nsub);
  const int64_t cb = cbounds[b], len = cbounds[b + 1] - cb;
  auto cut = [&](int k) {
    if (k == 0 || k == nsub) return cb + (k ? len : 0);
    const int64_t c = (cb + k * len / nsub) / 32 * 32;
    return c > cb ? c : cb;
  };
  const int lo = (int)cut(s), hi = (int)cut(s + 1);  // columns < 2^31
  const int64_t row0 = rt * C::ROWS;
  const int a0 = lo & ~31;
  const int64_t nb = lo < hi ? ((int64_t)hi - a0 + 31) / 32 : 0;
  float* const zbuf = smem + 2 * C::SLICE;

  double q[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (wave < 4) {
    u32x4 xh[C::KC], xm[C::KC], xl[C::KC];
    const bool in = load_x<RP>(xh, xm, xl, X, rows, row0, wave, lane >> 5, lane & 31);
    produce<RP>(smem, split + (int64_t)a0 / 32 * (48 * RP), nb, -1, nullptr, xh, xm, xl, wave, lane);
    if (!in) bad = 1;
  } else {
    __builtin_amdgcn_s_setprio(3);
    if (tid == 256) bad = 0;
    const int cw = wave - 4, rg = cw / C::KS, cp = cw % C::KS;
    const int64_t row = row0 + 32 * rg + (lane & 31);
    Walk w{0, 0, INT_MAX, INT_MAX, 0.f, 0.f};
    if (row < rows) {
      int64_t l = rowptr[(int64_t)b * (rows + 1) + row];
      int64_t h = rowptr[(int64_t)b * (rows + 1) + row + 1];
      w.end = h;
      while (l < h) {
        const int64_t mid = (l + h) >> 1;
        if (idx[mid] < lo) l = mid + 1; else h = mid;
      }
      w.ptr = l;
      if (l < w.end) {
        w.c0 = idx[l];
        w.v0 = val[l];
      }
      if (l + 1 < w.end) {
        w.c1 = idx[l + 1];
        w.v1 = val[l + 1];
      }
    }
    int out = 0;
    for (int64_t k = lane; k < nb; k += 64) out |= bad_blocks[a0 / 32 + k];
    s3::lds_barrier();
    for (int64_t k = 0; k < nb; ++k) {
      s3::lds_barrier();
      if constexpr (C::SL == 2) s3::lds_barrier();
      // the tiles of block k are in LDS
      tile_terms<RP, METRICS>(q, w, zbuf + (int)(k & 1) * (4 * C::ZT), a0 + 32 * (int)k, lo, hi, rg,
                              cp, lane, idx, val);
    }
    if (out) bad = 1;
  }
  // the consumers' sums, in a fixed order; the panel blocks' LDS is free
  double* red = reinterpret_cast<double*>(smem);
  if (wave >= 4) {
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) q[k] += __shfl_xor(q[k], off, 64);
      if (lane == 0) red[4 * k + wave - 4] = q[k];
    }
  }
  wg_barrier();
  if (tid < NQ)
    partial[(int64_t)tid * gridDim.x + logical] =
        bad ? __builtin_nan("")
            : (red[4 * tid] + red[4 * tid + 1]) + (red[4 * tid + 2] + red[4 * tid + 3]);
}

template <int RP>
static hipError_t objective_t(const float* X, int64_t rows, const float* work, int64_t n,
                              const int64_t* cbounds, int nblk, int nsub, const int64_t* rowptr,
                              const int32_t* idx, const float* val, bool metrics, double* partial,
                              int64_t* npartial, hipStream_t st) {
  using C = Cfg<RP>;
  const int64_t row_tiles = (rows + C::ROWS - 1) / C::ROWS;
  const int64_t total = row_tiles * nblk * nsub;
  *npartial = total;
  if (total <= 0) return hipSuccess;
  if (total > 0x7fffffffLL) return hipErrorInvalidValue;
  const int* bad = reinterpret_cast<const int*>(work + blocks_of(n) * (48 * (int64_t)RP));
  if (metrics)
    hipLaunchKernelGGL((objective_split_kernel<RP, true>), dim3((unsigned)total), dim3(512), 0, st, X,
                       rows, work, bad, cbounds, nsub, rowptr, idx, val, row_tiles, partial);
  else
    hipLaunchKernelGGL((objective_split_kernel<RP, false>), dim3((unsigned)total), dim3(512), 0, st, X,
                       rows, work, bad, cbounds, nsub, rowptr, idx, val, row_tiles, partial);
  return hipGetLastError();
}

}  // namespace sw

bool objective_split_rank(int rp) { return rp >= 64 && rp <= 512 && rp % 64 == 0; }

hipError_t launch_objective_split(const float* X, int64_t rows, const float* P, int64_t n,
                                  const int64_t* cbounds, int nblk, int nsub, const int64_t* rowptr,
                                  const int32_t* idx, const float* val, int rp, bool metrics,
                                  float* work, double* partial, int64_t* npartial, hipStream_t st) {
  hipError_t e = launch_panel_split(P, n, rp, work, st);
  if (e != hipSuccess) return e;
#define CALL(R)                                                                                  \
  sw::objective_t<R>(X, rows, work, n, cbounds, nblk, nsub, rowptr, idx, val, metrics, partial, \
                     npartial, st)
  switch (rp) {
    case 64: return CALL(64);
    case 128: return CALL(128);
    case 192: return CALL(192);
    case 256: return CALL(256);
    case 320: return CALL(320);
    case 384: return CALL(384);
    case 448: return CALL(448);
    case 512: return CALL(512);
  }
#undef CALL
  return hipErrorInvalidValue;
}

}  // namespace nmd
