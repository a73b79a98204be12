// Rectified products with L = X P^T on bf16 MFMA of three-term splits (split3.h), for r_p a multiple
// of 64.
//
// A workgroup is four pairs of waves, one pair per SIMD.  A producer wave holds 32 rows of X (of
// KW columns) as split operands and streams v_mfma_f32_32x32x16_bf16 over 32-row panel blocks; it
// has no branch in its loop and hands each 32 x 32 tile of L to a consumer wave through LDS.
// The consumers do what is irregular: they find the positive entries of their tile one block
// later, while the producers are on the next block, so their branches and waits run beside the
// matrix instructions of the first product instead of between them.  At r_p > 128 the rank is cut
// in two (three terms of more columns would not fit a wave's registers): two producers share the
// rows of a tile and the consumer adds their halves.  At r_p >= 384 a panel block is loaded in two
// slices, half of each producer's columns at a time, so that two of them fit the LDS.
//
// The split panel is stored fragment by fragment as the producers' lanes read it, so that both the
// direct loads into LDS and the reads from it are plain runs of 1 KB.

#pragma once

#include "split3.h"

namespace nmd {
namespace sw {

using s3::floatx16;
using s3::mfma;
using s3::u32x4;

template <int RP_>
struct Cfg {
  static constexpr int RP = RP_;
  static constexpr int KS = RP > 128 ? 2 : 1;       // producers a tile's rank is cut over
  static constexpr int KW = RP / KS;                // columns of X a producer holds
  static constexpr int KC = KW / 16;                // its k chunks
  static constexpr int SL = RP >= 384 ? 2 : 1;      // slices of a panel block
  static constexpr int KCS = KC / SL;               // k chunks a producer takes of a slice
  static constexpr int RG = 4 / KS;                 // 32-row groups per workgroup
  static constexpr int ROWS = split_rows(RP);
  // Two consumers share a tile at KS = 2, each with half of its rows of X and all columns of Y: what a
  // live panel row costs is mostly finding it and its quads, not the columns.
  static constexpr int XR = 32 / KS;                // rows of X a consumer takes
  static constexpr int NQ = XR / 4;                 // quads of them
  static constexpr int GC = RP / 64;                // columns of Y per lane
  static constexpr int WGS = RP <= 64 ? 2 : 1;      // workgroups sharing a CU
  static constexpr int PIECES = KS * KCS * 3;       // 1 KB direct loads of a slice
  static constexpr int SLICE = 256 * PIECES;        // its floats
  static constexpr int ZT = 1024;                   // floats of a producer's L tile
  static constexpr int LDS = 2 * SLICE + 2 * 4 * ZT;
  static_assert(RP % 64 == 0 && RP <= 512 && KC % SL == 0 && LDS * 4 + 64 <= 160 * 1024 &&
                ROWS == 32 * RG, "shape");
};

// This wave's memory operations are done, then s_barrier; the empty asm statements keep the
// compiler from moving memory accesses across it.
__device__ __forceinline__ void wg_barrier() {
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// A flag in LDS, wave-uniform.
__device__ __forceinline__ bool seen(const int* flag) {
  return __builtin_amdgcn_readfirstlane(*(volatile const int*)flag) != 0;
}

// The rows of X a producer holds: lane (h, l32) holds row l32, columns 16 t + 8 h .. + 7 of chunk t.
// Returns false if a value lies outside the splits' range.
template <int RP>
__device__ __forceinline__ bool load_x(u32x4 (&xh)[Cfg<RP>::KC], u32x4 (&xm)[Cfg<RP>::KC],
                                       u32x4 (&xl)[Cfg<RP>::KC], const float* __restrict__ X,
                                       int64_t rows, int64_t row0, int wave, int h, int l32) {
  using C = Cfg<RP>;
  const int rg = wave / C::KS, kp = wave % C::KS;
  const int64_t row = row0 + 32 * rg + l32;
  const bool in = row < rows;  // a row past the end reads the last one and counts zero
  const float* base = X + (in ? row : rows - 1) * RP + kp * C::KW + 8 * h;
  s3::Range range;
  // a few chunks' loads in flight: all of them and the splits would not fit the registers
  constexpr int U = C::KC > 10 || C::WGS > 1 ? 2 : 4;
#pragma unroll
  for (int t0 = 0; t0 < C::KC; t0 += U) {
    float4 v[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (t0 + u >= C::KC) continue;
      v[u][0] = *reinterpret_cast<const float4*>(base + 16 * (t0 + u));
      v[u][1] = *reinterpret_cast<const float4*>(base + 16 * (t0 + u) + 4);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u;
      if (t >= C::KC) continue;
      const float4 a = v[u][0], b = v[u][1];
      const float x[8] = {in ? a.x : 0.f, in ? a.y : 0.f, in ? a.z : 0.f, in ? a.w : 0.f,
                          in ? b.x : 0.f, in ? b.y : 0.f, in ? b.z : 0.f, in ? b.w : 0.f};
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
    range.settle();
    __builtin_amdgcn_sched_barrier(0);
  }
  return !range.outside();
}

// Starts direct load u of producer `wave` (pieces wave, wave + 4, ...) from the slice at `src` into
// the LDS slice at `dst`.
template <int RP>
__device__ __forceinline__ void load_part(float* dst, const float* src, int u, int wave, int lane) {
  using C = Cfg<RP>;
  const int piece = wave + 4 * u;
  if (C::PIECES % 4 != 0 && piece >= C::PIECES) return;
  const char* from = reinterpret_cast<const char*>(src + 256 * piece);
  asm("" : "+s"(from));  // the uniform part stays in scalar registers, the lane's is 32 bits
  __builtin_amdgcn_global_load_lds((glb_void*)(from + (unsigned)(16 * lane)),
                                   (lds_void*)(dst + 256 * piece), 16, 0, 0);
}

// Adds slice S of a block to the tile of L, transposed: lane (h, l32), register v holds row l32 of
// the group and panel row 8 (v / 4) + 4 h + v % 4 of the block.  With `next`, this wave's share of
// a coming slice's direct loads into `nxt` is issued between the first MFMAs, two per chunk (issued
// back to back they block the wave for about 50 cycles each; spread over the whole slice the last
// ones are still in flight at the barrier).  The restrict qualifiers tell the compiler that the
// reads of `slice` do not depend on the loads in flight.  The small products have a chain of their
// own, so that the main sums round once per sixteen products.
template <int RP, int S>
__device__ __forceinline__ void l_slice(floatx16& acc, floatx16& low, const float* __restrict__ slice,
                                        float* __restrict__ nxt, const float* __restrict__ src,
                                        bool next, const u32x4 (&xh)[Cfg<RP>::KC],
                                        const u32x4 (&xm)[Cfg<RP>::KC],
                                        const u32x4 (&xl)[Cfg<RP>::KC], int wave, int lane) {
  using C = Cfg<RP>;
  constexpr int KCS = C::KCS;
  constexpr int LPW = (C::PIECES + 3) / 4;
  // chunks read ahead of their MFMAs (one where X takes three quarters of the registers)
  constexpr int LA = C::KC > 10 ? 1 : 2;
  const u32x4* pr = reinterpret_cast<const u32x4*>(slice + (wave % C::KS) * (KCS * 768)) + lane;
  u32x4 ph[KCS], pm[KCS], pl[KCS];
#pragma unroll
  for (int t = 0; t < (LA < KCS ? LA : KCS); ++t) {
    ph[t] = pr[192 * t];
    pm[t] = pr[192 * t + 64];
    pl[t] = pr[192 * t + 128];
  }
#pragma unroll
  for (int t = 0; t < KCS; ++t) {
    constexpr int X0 = S * KCS;
    if (t + LA < KCS) {
      ph[t + LA] = pr[192 * (t + LA)];
      pm[t + LA] = pr[192 * (t + LA) + 64];
      pl[t + LA] = pr[192 * (t + LA) + 128];
    }
    low = mfma(pl[t], xh[X0 + t], low);
    low = mfma(ph[t], xl[X0 + t], low);
    low = mfma(pm[t], xm[X0 + t], low);
    acc = mfma(ph[t], xh[X0 + t], acc);
    low = mfma(pm[t], xh[X0 + t], low);
    low = mfma(ph[t], xm[X0 + t], low);
    if (next) {
      constexpr int PER = LPW <= 2 * KCS ? 2 : 3;
#pragma unroll
      for (int u = 0; u < LPW; ++u)
        if (u / PER == t) load_part<RP>(nxt, src, u, wave, lane);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The producers' loop: nb panel blocks (split panel at `src`), one barrier before each slice and one
// after the last.  `stop` (if not negative): the barrier after which *quit may end the loop (every
// wave of the workgroup looks there; no load is in flight).  Returns false if it did.
template <int RP>
__device__ __forceinline__ bool produce(float* smem, const float* __restrict__ src, int64_t nb,
                                        int64_t stop, const int* quit, const u32x4 (&xh)[Cfg<RP>::KC],
                                        const u32x4 (&xm)[Cfg<RP>::KC],
                                        const u32x4 (&xl)[Cfg<RP>::KC], int wave, int lane) {
  using C = Cfg<RP>;
  float* zbase = smem + 2 * C::SLICE + wave * C::ZT + 4 * lane;
  if (nb > 0) {
#pragma unroll
    for (int u = 0; u < (C::PIECES + 3) / 4; ++u) load_part<RP>(smem, src, u, wave, lane);
  }
  int buf = 0;
  for (int64_t b = 0; b < nb; ++b) {
    floatx16 acc, low;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = low[v] = 0.f;
    wg_barrier();
    if (C::SL * b == stop && seen(quit)) return false;
    src += C::SLICE;
    l_slice<RP, 0>(acc, low, smem + buf * C::SLICE, smem + (buf ^ 1) * C::SLICE, src,
                   C::SL == 2 || b + 1 < nb, xh, xm, xl, wave, lane);
    buf ^= 1;
    if constexpr (C::SL == 2) {
      wg_barrier();
      if (C::SL * b + 1 == stop && seen(quit)) return false;
      src += C::SLICE;
      l_slice<RP, 1>(acc, low, smem + buf * C::SLICE, smem + (buf ^ 1) * C::SLICE, src, b + 1 < nb, xh,
                     xm, xl, wave, lane);
      buf ^= 1;
    }
    const floatx16 l = acc + low;
    float* z = zbase + (int)(b & 1) * (4 * C::ZT);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      *reinterpret_cast<float4*>(z + 256 * u) =
          make_float4(l[4 * u], l[4 * u + 1], l[4 * u + 2], l[4 * u + 3]);
  }
  wg_barrier();
  return true;
}

// The consumer's copy of the L tile of a block (the halves of the rank added).
template <int RP>
__device__ __forceinline__ void read_tile(float (&z)[16], const float* zt, int rg, int lane) {
  using C = Cfg<RP>;
  const float* src = zt + rg * C::KS * C::ZT + 4 * lane;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    float4 a = *reinterpret_cast<const float4*>(src + 256 * u);
    if constexpr (C::KS == 2) {
      const float4 b = *reinterpret_cast<const float4*>(src + C::ZT + 256 * u);
      a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
    }
    z[4 * u] = a.x; z[4 * u + 1] = a.y; z[4 * u + 2] = a.z; z[4 * u + 3] = a.w;
  }
}

// The panel rows with a positive entry in a tile (bit j: row j of the block), wave-uniform; a
// positive NaN or a -0 sets its bit too.  With KS = 2 among the rows of X 16 cp .. + 15 alone.  Bit v
// of a lane's mask is register v; the masks of each half of the wave are combined, and their groups of
// four bits interleaved (row 8 u + 4 h + c is register 4 u + c of half h).
template <int KS>
__device__ __forceinline__ unsigned live_rows(const float (&z)[16], int cp) {
  unsigned m = 0;
#pragma unroll
  for (int v = 15; v >= 0; --v) m = __builtin_amdgcn_alignbit(m, 0u - __float_as_uint(z[v]), 31);
  m |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x111, 0xf, 0xf, true);  // row_shr:1
  m |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x112, 0xf, 0xf, true);  // row_shr:2
  m |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x114, 0xf, 0xf, true);  // row_shr:4
  m |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x118, 0xf, 0xf, true);  // row_shr:8
  unsigned lo, hi;  // lane 16 k + 15 has its sixteen lanes'
  if constexpr (KS == 2) {
    lo = (unsigned)__builtin_amdgcn_readlane((int)m, 16 * cp + 15);
    hi = (unsigned)__builtin_amdgcn_readlane((int)m, 16 * cp + 47);
  } else {
    lo = (unsigned)(__builtin_amdgcn_readlane((int)m, 15) | __builtin_amdgcn_readlane((int)m, 31));
    hi = (unsigned)(__builtin_amdgcn_readlane((int)m, 47) | __builtin_amdgcn_readlane((int)m, 63));
  }
  const unsigned a = (lo | (lo << 8)) & 0x00ff00ffu, b = (hi | (hi << 8)) & 0x00ff00ffu;
  return ((a | (a << 4)) & 0x0f0f0f0fu) | (((b | (b << 4)) & 0x0f0f0f0fu) << 4);
}

// The work area of a panel: its split copy in whole 32-row blocks (rows past the panel are zero, so
// their L is zero), then one int per block: whether a value lies outside the splits' range.
// Fragment (block, slice, kp, t of KCS), term k (h, m, l) is 64 lanes of 16 bytes at ((((block SL +
// slice) KS + kp) KCS + t) 3 + k) 64: lane (h, l32) holds row l32, columns kp KW + 16 (slice KCS +
// t) + 8 h .. + 7.
inline int64_t blocks_of(int64_t blk) { return (blk + 31) / 32; }
inline int64_t work_floats(int64_t blk, int rp) { return blocks_of(blk) * (48 * (int64_t)rp + 1); }

}  // namespace sw
}  // namespace nmd
