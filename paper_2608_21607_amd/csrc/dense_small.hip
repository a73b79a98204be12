// The dense contraction Y = sgn max(0, X P^T) P at r_p <= 64, both products on bf16 MFMA of
// three-term splits (split3.h), which hold every operand whole.
//
// A wave holds 32 rows of X as split operands and takes the panel 32 rows at a time: L^T = P X^T
// as 32 x 32 tiles, so that a lane's sixteen entries of L belong to one row of X and are, in pairs of
// registers, already the operand of the second product Y^T += P^T max(0, L)^T.  The rectified
// entries, fp32 as they come, are split again.  Both products keep the small terms in accumulators
// of their own.
//
// The workgroup's eight waves share the panel through LDS: each thread reads four fp32 values
// a block ahead, splits them and writes them row-major to the other buffer.  The first product
// reads the rows as they lie, the second reads them transposed (ds_read_b64_tr_b16), so there is
// one copy and no pass over the panel before the launch.  Rows are padded by 16 bytes: sixteen rows'
// 16-byte chunks fall on distinct banks.
//
// What bounds it: the bf16 matrix rate and the vector work beside it (48 MFMAs a wave and 32 x 32 tile
// at r_p = 64); at r_p = 16 the vector work.  250000 x 2500, r = 64, half of L positive: 0.76 ms, 210
// TFLOP/s of the two products (1260 of bf16), against 1.21 ms of fp32 MFMA; 60000 x 8192, r = 48 / 32 /
// 16 0.54 / 0.34 / 0.26 ms against 0.82 / 0.58 / 0.37.  Two-term f16 splits with a scale per row took
// 0.55 ms at the first shape, but lost columns far below their row's largest (10^-2 of a column of Y at
// 2^-32) and the last bit of a quarter of the values.  The sums of the second product are taken in
// chains of kChain panel rows.  Error against fp64 at the first shape 5.9e-8 (fp32 MFMA: 5.2e-7).
//
// A workgroup whose rows or panel range hold an infinity, a NaN or a magnitude outside the splits'
// range, or whose sums overflow, computes its rows again in plain fp32.

#include "split3.h"

namespace nmd {
namespace fs {

using s3::floatx16;
using s3::mfma;
using s3::u32x2;
using s3::u32x4;
typedef short short4v __attribute__((ext_vector_type(4)));

template <int RP_>
struct Cfg {
  static constexpr int RP = RP_;
  static constexpr int WAVES = 8;
  static constexpr int ROWS = 32 * WAVES;
  static constexpr int LPR = RP <= 16 ? 4 : RP <= 32 ? 8 : 16;  // lanes that stage a panel row
  static constexpr int JB = 64 * WAVES / LPR;                   // panel rows per LDS block
  static constexpr int KC = RP / 16;                            // k chunks of the first product
  static constexpr int MT = (RP + 31) / 32;                     // column tiles of Y
  static constexpr int STR = 2 * RP + 16;                       // bytes of a row in LDS
  static constexpr int PLANE = JB * STR;                        // one term of the block
  static constexpr int BUF = 3 * PLANE;
  // registers of a column tile that hold columns of Y (half of the last tile's at 16 and 48)
  static constexpr int cols(int mt) { return 32 * mt + 16 < RP ? 16 : 8; }
};

constexpr int kChain = 256;  // panel rows per accumulator chain of the second product

// Four columns of 4 consecutive panel rows transposed: lane (l % 16) of a 16-lane group names four
// halves of row (l % 16) / 4 and receives the four rows' halves of column l % 16.
__device__ __forceinline__ u32x2 read_tr(const char* p) {
  typedef __attribute__((address_space(3))) short4v lds_short4;
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)p));
}

// One thread's share of a panel block: row tid / LPR, columns 4 (tid % LPR) .. + 3.
template <int RP>
__device__ __forceinline__ float4 fetch(const float* __restrict__ P, int64_t j0, int64_t jb1, int tid) {
  using C = Cfg<RP>;
  const int64_t j = j0 + tid / C::LPR;
  const int g = tid % C::LPR;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (j < jb1 && 4 * g < RP) v = *reinterpret_cast<const float4*>(P + j * RP + 4 * g);
  return v;
}

template <int RP>
__device__ __forceinline__ void stash(char* buf, float4 v, s3::Range& range, int tid) {
  using C = Cfg<RP>;
  const int j = tid / C::LPR, g = tid % C::LPR;
  range.see(v.x);
  range.see(v.y);
  range.see(v.z);
  range.see(v.w);
  u32x2 t[3];
  unsigned h, m, l;
  s3::split(v.x, v.y, h, m, l);
  t[0][0] = h; t[1][0] = m; t[2][0] = l;
  s3::split(v.z, v.w, h, m, l);
  t[0][1] = h; t[1][1] = m; t[2][1] = l;
  if (4 * g < RP) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      *reinterpret_cast<u32x2*>(buf + k * C::PLANE + j * C::STR + 8 * g) = t[k];
  }
}

// The workgroup's rows in plain fp32, for inputs outside the splits' range.  Entries of L that are
// not above zero (NaN included) add nothing.
template <int RP>
__device__ __noinline__ void plain_rows(const float* __restrict__ X, int64_t rows,
                                        const float* __restrict__ P, int64_t jb0, int64_t jb1,
                                        float* __restrict__ Y, int64_t row0, float sgn, int tid) {
  const int64_t row = row0 + (tid >> 1);
  const int k0 = (tid & 1) * (RP / 2);
  if (row >= rows) return;
  float y[RP / 2];
#pragma unroll
  for (int k = 0; k < RP / 2; ++k) y[k] = 0.f;
  for (int64_t j = jb0; j < jb1; ++j) {
    float l = 0.f;
    for (int k = 0; k < RP; ++k) l = fmaf(X[row * RP + k], P[j * RP + k], l);
    if (l > 0.f)
#pragma unroll
      for (int k = 0; k < RP / 2; ++k) y[k] = fmaf(l, P[j * RP + k0 + k], y[k]);
  }
#pragma unroll
  for (int k = 0; k < RP / 2; ++k) Y[row * RP + k0 + k] = sgn * y[k];
}

template <int RP>
__global__ __launch_bounds__(512, RP <= 16 ? 4 : 2) void dense_small_kernel(
    const float* __restrict__ X, int64_t rows, const float* __restrict__ P, int64_t blk,
    float* __restrict__ Ypart, int64_t y_stride, int nsplit, int64_t row_tiles, float sgn,
    unsigned long long* __restrict__ counts) {
  using C = Cfg<RP>;
  __shared__ __attribute__((aligned(16))) char smem[2 * C::BUF];
  __shared__ int bad;
  __shared__ unsigned total;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, l32 = lane & 31;

  const int64_t logical = xcd_logical(blockIdx.x, (int64_t)gridDim.x);
  const int s = (int)(logical / row_tiles);
  const int64_t rt = logical - (int64_t)s * row_tiles;
  const int64_t jb0 = (int64_t)s * blk / nsplit;
  const int64_t jb1 = (int64_t)(s + 1) * blk / nsplit;
  const int64_t row0 = rt * C::ROWS;
  const int64_t row = row0 + 32 * wave + l32;

  float4 next = fetch<RP>(P, jb0, jb1, tid);
  s3::Range range;
  if (tid == 0) bad = 0, total = 0;

  // the wave's rows of X: lane (h, l32) holds row l32, columns 16 t + 8 h .. + 7 of chunk t
  u32x4 xh[C::KC], xm[C::KC], xl[C::KC];
#pragma unroll
  for (int t = 0; t < C::KC; ++t) {
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    if (row < rows) {
      const float* src = X + row * RP + 16 * t + 8 * h;
      a = *reinterpret_cast<const float4*>(src);
      b = *reinterpret_cast<const float4*>(src + 4);
    }
    const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) range.see(x[e]);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      unsigned s0, s1, s2;
      s3::split(x[2 * w], x[2 * w + 1], s0, s1, s2);
      xh[t][w] = s0;
      xm[t][w] = s1;
      xl[t][w] = s2;
    }
  }

  // register 4 t + v of tile mt is column 32 mt + 8 t + 4 h + v; ys: the sums of yh, which starts
  // again every kChain panel rows, so that its roundings are those of a short chain
  floatx16 yh[C::MT], yl[C::MT];
  float ys[C::MT][16];
#pragma unroll
  for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
    for (int v = 0; v < 16; ++v) yh[mt][v] = yl[mt][v] = ys[mt][v] = 0.f;
  int chain = 0;
  unsigned slices = 0;

  stash<RP>(smem, next, range, tid);
  next = fetch<RP>(P, jb0 + C::JB, jb1, tid);
  s3::lds_barrier();

  // this lane's offsets in a block: its row of the first product, its four entries of the second
  // (at r_p = 16 and 48 the last tile's upper columns repeat the lower: their sums are not stored)
  const int at1 = l32 * C::STR + 16 * h;
  const int at2 = (4 * h + ((lane & 15) >> 2)) * C::STR + 8 * (lane & 3);
  const int up = 32 * ((lane >> 4) & 1);

  int cur = 0;
  for (int64_t j0 = jb0; j0 < jb1; j0 += C::JB) {
    const char* buf = smem + cur * C::BUF;
    if (j0 + C::JB < jb1) {
      stash<RP>(smem + (cur ^ 1) * C::BUF, next, range, tid);
      next = fetch<RP>(P, j0 + 2 * C::JB, jb1, tid);
    }
    const int64_t left = jb1 - j0;
    const int subs = left >= C::JB ? C::JB / 32 : (int)((left + 31) / 32);
    for (int sub = 0; sub < subs; ++sub) {
      const char* tile = buf + 32 * sub * C::STR;
      floatx16 acc, low;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = low[v] = 0.f;
#pragma unroll
      for (int t = 0; t < C::KC; ++t) {
        const u32x4 ph = *reinterpret_cast<const u32x4*>(tile + at1 + 32 * t);
        const u32x4 pm = *reinterpret_cast<const u32x4*>(tile + C::PLANE + at1 + 32 * t);
        const u32x4 pl = *reinterpret_cast<const u32x4*>(tile + 2 * C::PLANE + at1 + 32 * t);
        acc = mfma(ph, xh[t], acc);
        low = mfma(ph, xl[t], low);
        low = mfma(pl, xh[t], low);
        low = mfma(pm, xm[t], low);
        low = mfma(ph, xm[t], low);
        low = mfma(pm, xh[t], low);
      }
      // u: entries of max(0, L); register 4 t + v is panel row 8 t + 4 h + v
      float u[16], top[2] = {0.f, 0.f};
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        u[v] = fmaxf(acc[v] + low[v], 0.f);
        top[v >> 3] = fmaxf(top[v >> 3], u[v]);
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        // the chunk's 16 panel rows x the wave's 32 rows: skipped where L has no positive entry
        const unsigned long long live = __ballot(top[c] > 0.f);
        if (live == 0) continue;
        slices += 4u * (((live & 0x0000ffff0000ffffull) != 0) + ((live & 0xffff0000ffff0000ull) != 0));
        u32x4 zh, zm, zl;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          unsigned s0, s1, s2;
          s3::split(u[8 * c + 2 * w], u[8 * c + 2 * w + 1], s0, s1, s2);
          zh[w] = s0;
          zm[w] = s1;
          zl[w] = s2;
        }
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt) {
          const char* p = tile + at2 + 16 * c * C::STR + 64 * mt + (32 * mt + 16 < RP ? up : 0);
          u32x4 q[3];
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const u32x2 a = read_tr(p + k * C::PLANE), b = read_tr(p + k * C::PLANE + 8 * C::STR);
            q[k] = u32x4{a[0], a[1], b[0], b[1]};
          }
          yh[mt] = mfma(q[0], zh, yh[mt]);
          yl[mt] = mfma(q[0], zl, yl[mt]);
          yl[mt] = mfma(q[2], zh, yl[mt]);
          yl[mt] = mfma(q[1], zm, yl[mt]);
          yl[mt] = mfma(q[0], zm, yl[mt]);
          yl[mt] = mfma(q[1], zh, yl[mt]);
        }
      }
    }
    if ((chain += C::JB) == kChain) {
      chain = 0;
#pragma unroll
      for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          if (v < C::cols(mt)) ys[mt][v] += yh[mt][v];
          yh[mt][v] = 0.f;
        }
    }
    cur ^= 1;
    s3::lds_barrier();
  }

  float* Y = Ypart + (int64_t)s * y_stride;
  bool again = range.outside();
#pragma unroll
  for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
    for (int v = 0; v < C::cols(mt); ++v) {
      ys[mt][v] = sgn * (ys[mt][v] + (yh[mt][v] + yl[mt][v]));
      again |= !isfinite(ys[mt][v]);
    }
  if (again) bad = 1;
  if (lane == 0 && slices) atomicAdd(&total, slices);
  __syncthreads();
  if (bad) {
    plain_rows<RP>(X, rows, P, jb0, jb1, Y, row0, sgn, tid);
  } else if (row < rows) {
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (32 * mt + 8 * t < RP)
          *reinterpret_cast<float4*>(Y + row * RP + 32 * mt + 8 * t + 4 * h) =
              make_float4(ys[mt][4 * t], ys[mt][4 * t + 1], ys[mt][4 * t + 2], ys[mt][4 * t + 3]);
  }
  if (counts && tid == 0 && total) atomicAdd(counts, (unsigned long long)total);
}

template <int RP>
static hipError_t launch_t(const float* X, int64_t rows, const float* P, int64_t blk, float* Ypart,
                           int64_t y_stride, int nsplit, float sgn, unsigned long long* counts,
                           hipStream_t st) {
  const int64_t row_tiles = (rows + Cfg<RP>::ROWS - 1) / Cfg<RP>::ROWS;
  const int64_t total = row_tiles * nsplit;
  if (total <= 0) return hipSuccess;
  if (total > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((dense_small_kernel<RP>), dim3((unsigned)total), dim3(64 * Cfg<RP>::WAVES), 0,
                     st, X, rows, P, blk, Ypart, y_stride, nsplit, row_tiles, sgn, counts);
  return hipGetLastError();
}

}  // namespace fs

int dense_small_rows_per_wg() { return fs::Cfg<64>::ROWS; }

hipError_t dense_small_wgs_per_cu(int rp, int* out) {
#define CALL(R) hipOccupancyMaxActiveBlocksPerMultiprocessor(out, fs::dense_small_kernel<R>, 512, 0)
  switch (rp) {
    case 16: return CALL(16);
    case 32: return CALL(32);
    case 48: return CALL(48);
    case 64: return CALL(64);
  }
#undef CALL
  return hipErrorInvalidValue;
}

hipError_t launch_dense_small(const float* X, int64_t rows, const float* P, int64_t blk, int rp,
                              float* Ypart, int64_t y_stride, int nsplit, float sgn,
                              unsigned long long* counts, hipStream_t st) {
#define CALL(R) fs::launch_t<R>(X, rows, P, blk, Ypart, y_stride, nsplit, sgn, counts, st)
  switch (rp) {
    case 16: return CALL(16);
    case 32: return CALL(32);
    case 48: return CALL(48);
    case 64: return CALL(64);
  }
#undef CALL
  return hipErrorInvalidValue;
}

}  // namespace nmd
