// The rectified contraction Y = sgn * max(0, X P^T) P with its first product on bf16 MFMA of
// three-term splits (split_wide.h), for r_p >= 128; the second product is fp32, on the panel's own
// rows, for the positive entries alone.
//
// What bounds it: at no positive entry the matrix rate, 1.0 to 1.1 PFLOP/s of bf16 (independent MFMAs on
// random operands 1.76 at the card's power limit; without the direct loads 15% less time, without the
// consumers 5%); with entries the consumers, whose work per live panel row is a chain of scalar tests.
// 8192 panel rows, none / 0.5% of L positive, ms: 139255 rows, r_p = 256 3.2 / 3.6 (fp32 kernel 4.5 /
// 5.2); 60000 rows, 128 0.70 / 0.99 (1.14 / 1.38), 192 1.20 / 1.42 (1.81 / 2.23), 320 1.83 / 1.97 (3.29 /
// 4.10), 384 2.14 / 2.57 (3.83 / 4.91), 448 2.41 / 2.81 (4.42 / 5.67); 125000 rows, 512 5.5 / 6.7 (9.0 /
// 10.0).  With two-term f16 splits the first product took half of this, but lost the operands' last
// bits and small columns.

#include "split_wide.h"

namespace nmd {
namespace sw {

// The split copy of a panel: a workgroup per 32-row block, its waves taking the block's 16-column
// chunks in turn.  `bad` receives an int per block: 1 if a value lies outside the splits' range.
template <int RP>
__global__ __launch_bounds__(256) void panel_split_kernel(const float* __restrict__ P, int64_t blk,
                                                          u32x4* __restrict__ split,
                                                          int* __restrict__ bad) {
  using C = Cfg<RP>;
  __shared__ int any;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t block = blockIdx.x;
  const int64_t row = 32 * block + (lane & 31);
  if (threadIdx.x == 0) any = 0;
  __syncthreads();
  s3::Range range;
  for (int g = wave; g < RP / 16; g += 4) {
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    if (row < blk) {
      const float* src = P + row * RP + 16 * g + 8 * (lane >> 5);
      a = *reinterpret_cast<const float4*>(src);
      b = *reinterpret_cast<const float4*>(src + 4);
    }
    const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) range.see(x[e]);
    u32x4 q[3];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      unsigned s0, s1, s2;
      s3::split(x[2 * w], x[2 * w + 1], s0, s1, s2);
      q[0][w] = s0;
      q[1][w] = s1;
      q[2][w] = s2;
    }
    const int kp = g / C::KC, t = g % C::KC;
    const int64_t frag = ((block * C::SL + t / C::KCS) * C::KS + kp) * C::KCS + t % C::KCS;
#pragma unroll
    for (int k = 0; k < 3; ++k) split[(frag * 3 + k) * 64 + lane] = q[k];
  }
  if (range.outside()) any = 1;
  __syncthreads();
  if (threadIdx.x == 0) bad[block] = any;
}

// One panel row's second-product operands (with a NaN in X a row past the panel's end may look live:
// the panel's buffer has 256 rows of padding): its column of L (row l of the consumer's XR in the lanes
// l, l + XR, ...) and GC columns of the panel row per lane.
template <int GC>
struct LiveRow {
  float z0, z1;
  float p[GC];
};

template <int RP>
__device__ __forceinline__ LiveRow<Cfg<RP>::GC> fetch_row(int j, const float* zl,
                                                          const float* __restrict__ panel, int lane) {
  using C = Cfg<RP>;
  LiveRow<C::GC> r;
  const float* zs = zl + ((j >> 2) * 128 + (j & 3));
  r.z0 = zs[0];
  r.z1 = C::KS == 2 ? zs[C::ZT] : 0.f;
  const float* row = panel + j * RP + (unsigned)(C::GC * lane);
  if constexpr (C::GC % 4 == 0) {
#pragma unroll
    for (int g = 0; g < C::GC; g += 4) {
      const float4 a = *reinterpret_cast<const float4*>(row + g);
      r.p[g] = a.x; r.p[g + 1] = a.y; r.p[g + 2] = a.z; r.p[g + 3] = a.w;
    }
  } else if constexpr (C::GC % 2 == 0) {
#pragma unroll
    for (int g = 0; g < C::GC; g += 2) {
      const float2 a = *reinterpret_cast<const float2*>(row + g);
      r.p[g] = a.x; r.p[g + 1] = a.y;
    }
  } else {
#pragma unroll
    for (int g = 0; g < C::GC; ++g) r.p[g] = row[g];
  }
  return r;
}

template <int A, int NQ, int GC>
__device__ __forceinline__ void quad(floatx4 (&y)[NQ][GC], float z, const float (&p)[GC]) {
#pragma unroll
  for (int g = 0; g < GC; ++g)
    y[A][g] = __builtin_amdgcn_mfma_f32_4x4x1f32(z, p[g], y[A][g], 4, A, 0);
}

// quad<q> for the quads LO .. LO + N - 1 with a live row, by halving (a nested if per level: most
// rows have one live quad).
template <int LO, int N, int NQ, int GC>
__device__ __forceinline__ void live_quads(floatx4 (&y)[NQ][GC], float z, const float (&p)[GC],
                                           unsigned live) {
  if constexpr (N == 1) {
    if (live & (15u << (4 * LO))) quad<LO>(y, z, p);
  } else {
    constexpr unsigned mask = (N == 8 ? 0xffffffffu : (1u << (4 * N % 32)) - 1u) << (4 * LO);
    if (N == NQ || (live & mask)) {
      live_quads<LO, N / 2>(y, z, p, live);
      live_quads<LO + N / 2, N / 2>(y, z, p, live);
    }
  }
}

// Adds the row's positive entries: per quad of rows holding one, GC v_mfma_f32_4x4x1 whose A
// operand is the quad's four values broadcast to all blocks (CBSZ = 4, ABID = quad).  y[a][g],
// register v, lane l holds Y[4 a + v][GC l + g].
template <int NQ, int GC>
__device__ __forceinline__ unsigned add_row(floatx4 (&y)[NQ][GC], const LiveRow<GC>& r) {
  const float z = fmaxf(r.z0 + r.z1, 0.f);
  const unsigned live = (unsigned)__ballot(z > 0.f) & (NQ == 8 ? 0xffffffffu : 0xffffu);
  live_quads<0, NQ>(y, z, r.p, live);
  return __builtin_popcount(live);
}

// A consumer's rows in flight: up to DEEP live panel rows of a block are requested together and
// added while the producers work on the next block, so that a block with few entries waits for no
// load of its own.  (Graph sweep, r = 256, 0.4% positive, where a consumer meets two rows a block: six
// 136 ms of contraction, three 131, by their untaken branches.)

template <int RP>
struct Pending {
  static constexpr int DEEP = Cfg<RP>::KS == 2 ? 3 : 6;
  LiveRow<Cfg<RP>::GC> r[DEEP];
  int n = 0;

  __device__ __forceinline__ unsigned add(floatx4 (&y)[Cfg<RP>::NQ][Cfg<RP>::GC]) {
    unsigned entries = 0;
#pragma unroll
    for (int k = 0; k < DEEP; ++k)
      if (k < n) entries += add_row(y, r[k]);
    n = 0;
    return entries;
  }
  // takes rows off `rows` (n = 0 before)
  __device__ __forceinline__ void fetch(unsigned& rows, const float* zl, const float* panel, int lane) {
    const int have = __builtin_popcount(rows);
    n = have < DEEP ? have : DEEP;
#pragma unroll
    for (int k = 0; k < DEEP; ++k) {
      if (k < n) r[k] = fetch_row<RP>(__builtin_ctz(rows), zl, panel, lane);
      rows &= rows - 1;
    }
  }
};

// The share of positive entries beyond which a workgroup leaves its rows to the fp32 kernel, which
// takes them by slices at r_p other than 256 and 512 where a consumer pays for each.  Measured with L
// alike everywhere (8192 panel rows, 60000 rows; r_p = 256 139255, 512 125000), split / fp32 in ms:
//   r_p = 128  2.0% 1.80 / 1.93   3.0% 2.18 / 2.05   4.0% 2.50 / 2.13   50% 4.49 / 2.28
//         192  3.0% 2.93 / 3.25   6.0% 3.92 / 3.36   50% 7.23 / 3.44
//         256  3.0% 6.99 / 7.28   6.0% 9.36 / 8.20   50% 17.4 / 10.9
//         320   10% 5.28 / 5.51    16% 6.27 / 5.55   50% 7.73 / 5.57
//         384   10% 6.23 / 6.40    16% 7.30 / 6.44   50% 9.40 / 6.46
//         448   12% 6.92 / 7.44    16% 7.69 / 7.45   50% 9.81 / 7.51
//         512   16% 16.5 / 17.8    50% 20.9 / 20.5
// The line lies where the split kernel takes about 1.15 times as long: a few tiles on their own cost a
// whole workgroup's length behind it (guarded sweeps of 34814 x 34814, r = 200 with 1.8% positive:
// 16.6 ms of contraction with the line at 3.5%, 13.7 at 6% and without one).
constexpr float dense_from(int rp) {
  return rp <= 128 ? 0.045f : rp <= 256 ? 0.06f : rp <= 384 ? 0.16f : rp <= 448 ? 0.25f : 2.f;
}

// A workgroup that finds L dense stops, and one that met a value outside the splits' range or a sum
// that is not finite throws its result away: redo[split row_tiles + row tile] tells the fp32 kernel
// behind this one to form those rows.  Dense: more than `dense` of its entries positive in the first
// block, or two of 32 and more (not where the range has less than three).
template <int RP>
__global__ __launch_bounds__(512, 2 * Cfg<RP>::WGS) void dense_split_kernel(
    const float* __restrict__ X, int64_t rows, const float* __restrict__ P,
    const float* __restrict__ split, const int* __restrict__ bad_blocks, int64_t blk,
    float* __restrict__ Ypart, int64_t y_stride, int nsplit, int64_t row_tiles, float sgn,
    float dense, int* __restrict__ redo, unsigned long long* __restrict__ counts) {
  using C = Cfg<RP>;
  __shared__ __attribute__((aligned(16))) float smem[C::LDS];
  __shared__ int bad, quit;
  __shared__ unsigned positive;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // in launch order, so that neighbouring row tiles lie on different XCDs: where rows are sorted by
  // how many entries they have, a run of them per XCD made the first one's take longer (125000 x
  // 50000 word counts, r = 512 118 ms a sweep, 115 so)
  const int64_t logical = blockIdx.x;
  const int s = (int)(logical / row_tiles);
  const int64_t rt = logical - (int64_t)s * row_tiles;
  const int64_t jb0 = block_start(s, nsplit, blk);
  const int64_t jb1 = block_start(s + 1, nsplit, blk);
  const int64_t row0 = rt * C::ROWS;
  const int64_t nb = (jb1 - jb0 + 31) / 32;
  // the last block looked at for a dense L, and the barrier after which every wave looks at `quit`
  const int64_t look = nb < 3 ? -1 : nb < 32 ? 0 : 1;
  const int64_t stop = look < 0 ? -1 : (look + 1) * C::SL + 1;
  float* const zbuf = smem + 2 * C::SLICE;

  if (wave < 4) {
    u32x4 xh[C::KC], xm[C::KC], xl[C::KC];
    const bool in = load_x<RP>(xh, xm, xl, X, rows, row0, wave, lane >> 5, lane & 31);
    if (!produce<RP>(smem, split + jb0 / 32 * (48 * RP), nb, stop, &quit, xh, xm, xl, wave, lane))
      return;
    if (!in) bad = 1;
    wg_barrier();
    return;
  }

  __builtin_amdgcn_s_setprio(3);
  const int cw = wave - 4;
  const int rg = cw / C::KS, cp = cw % C::KS;
  if (tid == 256) bad = 0, quit = 0, positive = 0;
  floatx4 y[C::NQ][C::GC];
#pragma unroll
  for (int a = 0; a < C::NQ; ++a)
#pragma unroll
    for (int g = 0; g < C::GC; ++g) y[a][g] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int x0 = 32 * rg + C::XR * cp;  // the consumer's first row of the tile
  const float* prow = P + jb0 * RP;
  int out = 0;
  for (int64_t b = lane; b < nb; b += 64) out |= bad_blocks[jb0 / 32 + b];

  unsigned entries = 0, rest = 0;
  Pending<RP> pending;
  const float* zl = zbuf;  // of the block whose rows are left
  const float* panel = prow;
  auto add_rest = [&]() {
    while (rest) {
      entries += pending.add(y);
      pending.fetch(rest, zl, panel, lane);
    }
  };
  s3::lds_barrier();
  for (int64_t b = 0; b < nb; ++b) {
    s3::lds_barrier();
    if (b == look + 1 && look >= 0) {
      if (seen(&quit)) {
        if (tid == 256) redo[logical] = 1;
        return;
      }
    }
    if constexpr (C::SL == 2) {
      add_rest();  // of the block before
      s3::lds_barrier();
    }
    // the tiles of block b are in LDS
    const float* zt = zbuf + (int)(b & 1) * (4 * C::ZT);
    {
      float z[16];
      read_tile<RP>(z, zt, rg, lane);
      rest = live_rows<C::KS>(z, cp);
      if (b <= look) {
        const unsigned long long mine = C::KS == 2 ? 0x0000ffff0000ffffull << (16 * cp) : ~0ull;
        unsigned n = 0;
#pragma unroll
        for (int v = 0; v < 16; ++v) n += (unsigned)__popcll(__ballot(z[v] > 0.f) & mine);
        if (lane == 0) {
          const unsigned all = atomicAdd(&positive, n) + n;
          if ((float)all > dense * (float)((look + 1) * 32 * C::ROWS)) quit = 1;
        }
      }
    }
    entries += pending.add(y);
    zl = zt + rg * C::KS * C::ZT + 4 * (C::XR * cp + lane % C::XR);
    panel = prow + b * (32 * RP);
    pending.fetch(rest, zl, panel, lane);
    if constexpr (C::SL == 1) add_rest();
  }
  if constexpr (C::SL == 2) add_rest();
  entries += pending.add(y);

  bool finite = true;
#pragma unroll
  for (int a = 0; a < C::NQ; ++a)
#pragma unroll
    for (int g = 0; g < C::GC; ++g)
#pragma unroll
      for (int v = 0; v < 4; ++v) finite = finite && isfinite(y[a][g][v]);
  if (out || !finite) bad = 1;
  wg_barrier();
  const bool again = seen(&bad);
  if (tid == 256) redo[logical] = again;
  if (again) return;
  float* Y = Ypart + (int64_t)s * y_stride;
#pragma unroll
  for (int a = 0; a < C::NQ; ++a)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t row = row0 + x0 + 4 * a + v;
      if (row >= rows) continue;
      float* dst = &Y[row * RP + C::GC * lane];
      if constexpr (C::GC % 4 == 0) {
#pragma unroll
        for (int g = 0; g < C::GC; g += 4)
          *reinterpret_cast<float4*>(dst + g) = make_float4(sgn * y[a][g][v], sgn * y[a][g + 1][v],
                                                            sgn * y[a][g + 2][v], sgn * y[a][g + 3][v]);
      } else if constexpr (C::GC % 2 == 0) {
#pragma unroll
        for (int g = 0; g < C::GC; g += 2)
          *reinterpret_cast<float2*>(dst + g) = make_float2(sgn * y[a][g][v], sgn * y[a][g + 1][v]);
      } else {
#pragma unroll
        for (int g = 0; g < C::GC; ++g) dst[g] = sgn * y[a][g][v];
      }
    }
  if (counts && lane == 0 && entries) atomicAdd(counts + 1, (unsigned long long)entries);
}

template <int RP>
static hipError_t launch_t(const float* X, int64_t rows, const float* P, int64_t blk, float* work,
                           float* Ypart, int64_t y_stride, int nsplit, float sgn, float dense,
                           int* redo, unsigned long long* counts, hipStream_t st) {
  using C = Cfg<RP>;
  const int64_t row_tiles = (rows + C::ROWS - 1) / C::ROWS;
  const int64_t total = row_tiles * nsplit;
  if (total <= 0) return hipSuccess;
  if (total > 0x7fffffffLL) return hipErrorInvalidValue;
  const int* bad = reinterpret_cast<const int*>(work + blocks_of(blk) * (48 * (int64_t)RP));
  hipLaunchKernelGGL((dense_split_kernel<RP>), dim3((unsigned)total), dim3(512), 0, st, X, rows, P,
                     work, bad, blk, Ypart, y_stride, nsplit, row_tiles, sgn, dense, redo, counts);
  return hipGetLastError();
}

template <int RP>
static hipError_t split_t(const float* P, int64_t blk, float* work, hipStream_t st) {
  const int64_t nblk = blocks_of(blk);
  hipLaunchKernelGGL((panel_split_kernel<RP>), dim3((unsigned)nblk), dim3(256), 0, st, P, blk,
                     reinterpret_cast<u32x4*>(work),
                     reinterpret_cast<int*>(work + nblk * (48 * (int64_t)RP)));
  return hipGetLastError();
}

}  // namespace sw

bool split_rank(int rp) { return rp >= 128 && rp <= 512 && rp % 64 == 0; }
int64_t split_work_floats(int64_t blk, int rp) { return sw::work_floats(blk, rp); }
int split_rows_per_wg(int rp) { return split_rows(rp); }
int64_t split_block_start(int s, int nsplit, int64_t blk) { return block_start(s, nsplit, blk); }

hipError_t launch_panel_split(const float* P, int64_t blk, int rp, float* work, hipStream_t st) {
  switch (rp) {
    case 64: return sw::split_t<64>(P, blk, work, st);
    case 128: return sw::split_t<128>(P, blk, work, st);
    case 192: return sw::split_t<192>(P, blk, work, st);
    case 256: return sw::split_t<256>(P, blk, work, st);
    case 320: return sw::split_t<320>(P, blk, work, st);
    case 384: return sw::split_t<384>(P, blk, work, st);
    case 448: return sw::split_t<448>(P, blk, work, st);
    case 512: return sw::split_t<512>(P, blk, work, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_dense_split(const float* X, int64_t rows, const float* P, int64_t blk, int rp,
                              float* work, float* Ypart, int64_t y_stride, int nsplit, float sgn,
                              int* redo, unsigned long long* counts, hipStream_t st) {
  hipError_t e = launch_panel_split(P, blk, rp, work, st);
  if (e != hipSuccess) return e;
#define CALL(R)                                                                                    \
  sw::launch_t<R>(X, rows, P, blk, work, Ypart, y_stride, nsplit, sgn, sw::dense_from(R), redo, counts, st)
  switch (rp) {
    case 128: e = CALL(128); break;
    case 192: e = CALL(192); break;
    case 256: e = CALL(256); break;
    case 320: e = CALL(320); break;
    case 384: e = CALL(384); break;
    case 448: e = CALL(448); break;
    case 512: e = CALL(512); break;
    default: return hipErrorInvalidValue;
  }
#undef CALL
  if (e != hipSuccess) return e;
  // the fp32 kernel, for the rows of the workgroups that stopped
  return launch_dense(X, rows, P, blk, rp, Ypart, y_stride, nsplit, sgn, counts, redo, st);
}

}  // namespace nmd
