// Layout helpers: the caller's W (m x r) and H (r x n) <-> the padded panels A (m x rp) and
// B = H^T (n x rp) the kernels work on, plus a fill and an ordered fp64 reduction.

#include "nmd_internal.h"

namespace nmd {

// Both panels in one launch: units below `row_units` copy 256 elements of W (m x r) into A (m x rp,
// zeros beyond r), the others 32 x 32 tiles of H (r x n) through LDS into B (n x rp).
__global__ __launch_bounds__(256) void load_panels_kernel(const float* __restrict__ W, int64_t m,
                                                          const float* __restrict__ H, int64_t n,
                                                          int r, int rp, float* __restrict__ A,
                                                          float* __restrict__ B, int64_t row_units,
                                                          int64_t col_tiles, int64_t units) {
  __shared__ float t[32][33];
  for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
    if (u < row_units) {
      const int64_t e = u * 256 + threadIdx.x;
      if (e >= m * rp) continue;
      const int64_t i = e / rp;
      const int c = (int)(e - i * rp);
      A[e] = c < r ? W[i * r + c] : 0.f;
      continue;
    }
    const int64_t g = u - row_units;
    const int64_t j0 = (g % col_tiles) * 32;
    const int c0 = (int)(g / col_tiles) * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 256 threads: 32 x 8
    __syncthreads();  // the tile before has been read
    for (int k = ty; k < 32; k += 8) {
      const int c = c0 + k;
      const int64_t j = j0 + tx;
      t[k][tx] = (c < r && j < n) ? H[(int64_t)c * n + j] : 0.f;
    }
    __syncthreads();
    for (int k = ty; k < 32; k += 8) {
      const int64_t j = j0 + k;
      const int c = c0 + tx;
      if (j < n && c < rp) B[j * rp + c] = t[tx][k];
    }
  }
}

// The way back; the first thread also writes the status words to pinned host memory (host_status
// may be NULL), which saves a copy of eight bytes and its wait.
__global__ __launch_bounds__(256) void store_panels_kernel(const float* __restrict__ A, int64_t m,
                                                           const float* __restrict__ B, int64_t n,
                                                           int r, int rp, float* __restrict__ W,
                                                           float* __restrict__ H, int64_t row_units,
                                                           int64_t col_tiles, int64_t units,
                                                           const int* status, int* host_status) {
  __shared__ float t[32][33];
  if (blockIdx.x == 0 && threadIdx.x == 0 && host_status) {
    host_status[0] = status[0];
    host_status[1] = status[1];
  }
  for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
    if (u < row_units) {
      const int64_t e = u * 256 + threadIdx.x;
      if (e >= m * r) continue;
      const int64_t i = e / r;
      const int c = (int)(e - i * r);
      W[e] = A[i * rp + c];
      continue;
    }
    const int64_t g = u - row_units;
    const int64_t j0 = (g % col_tiles) * 32;
    const int c0 = (int)(g / col_tiles) * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    __syncthreads();  // the tile before has been read
    for (int k = ty; k < 32; k += 8) {
      const int64_t j = j0 + k;
      const int c = c0 + tx;
      t[k][tx] = (j < n && c < rp) ? B[j * rp + c] : 0.f;
    }
    __syncthreads();
    for (int k = ty; k < 32; k += 8) {
      const int c = c0 + k;
      const int64_t j = j0 + tx;
      if (c < r && j < n) H[(int64_t)c * n + j] = t[tx][k];
    }
  }
}

// Zeroes two buffers and sets the status words to "no failure".
__global__ __launch_bounds__(256) void reset_kernel(float4* __restrict__ a, int64_t na,
                                                    float4* __restrict__ b, int64_t nb,
                                                    int* status) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    status[0] = 0;
    status[1] = 0x7f7f7f7f;
  }
  const int64_t step = (int64_t)gridDim.x * 256;
  const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < na; e += step) a[e] = z;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < nb; e += step) b[e] = z;
}

__global__ void zero_kernel(float* __restrict__ p, int64_t count) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < count) p[e] = 0.f;
}

// A copy that does nothing once the status word holds a failure (the snapshot of the factors
// before a sweep must not be overwritten by the state after a sweep that was rejected).
__global__ void guarded_copy_kernel(const float4* __restrict__ src, float4* __restrict__ dst,
                                    int64_t n4, const int* status) {
  if (*(volatile const int*)status != 0) return;
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < n4) dst[e] = src[e];
}

__global__ void guarded_copy_tail_kernel(const float* __restrict__ src, float* __restrict__ dst,
                                         int64_t begin, int64_t count, const int* status) {
  if (*(volatile const int*)status != 0) return;
  const int64_t e = begin + (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < count) dst[e] = src[e];
}

__global__ void guard_kernel(const double* __restrict__ q_old, const double* __restrict__ q_new,
                             double tol2, int* status, int step_id) {
  if (threadIdx.x != 0 || *(volatile const int*)status != 0) return;
  if (!(*q_new <= tol2 * *q_old)) {
    flag_status(status, STATUS_RISE, step_id);
  }
}

// Workgroup k: sum k of gridDim.x, per-thread strided partial sums, then a fixed-order tree.
__global__ __launch_bounds__(1024) void sum_kernel(const double* __restrict__ partial,
                                                   int64_t count, double* __restrict__ out,
                                                   int* is_nan, const int* when) {
  __shared__ double red[1024];
  if (when && *when == 0) return;
  const double* p = partial + (int64_t)blockIdx.x * count;
  double s = 0.0;
  for (int64_t e = threadIdx.x; e < count; e += 1024) s += p[e];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = 512; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[blockIdx.x] = red[0];
    if (is_nan && blockIdx.x == 0) *is_nan = isnan(red[0]);
  }
}

static inline unsigned blocks(int64_t n) { return (unsigned)((n + 255) / 256); }

// The panel copies' units: 256 elements of the rows, then 32 x 32 tiles of H.  A launch holds fewer
// than 2^32 threads, which both panels together may need more of (each alone had a launch before).
struct PanelUnits {
  int64_t rows, tiles, all;
  unsigned wgs;
  PanelUnits(int64_t row_elems, int64_t n, int rank)
      : rows((row_elems + 255) / 256), tiles((n + 31) / 32), all(rows + tiles * ((rank + 31) / 32)),
        wgs((unsigned)(all < (1 << 23) ? all : 1 << 23)) {}
};

hipError_t launch_load_panels(const float* W, int64_t m, const float* H, int64_t n, int r, int rp,
                              float* A, float* B, hipStream_t st) {
  const PanelUnits u(m * rp, n, rp);
  hipLaunchKernelGGL(load_panels_kernel, dim3(u.wgs), dim3(256), 0, st, W, m, H, n, r, rp, A, B, u.rows,
                     u.tiles, u.all);
  return hipGetLastError();
}

hipError_t launch_store_panels(const float* A, int64_t m, const float* B, int64_t n, int r, int rp,
                               float* W, float* H, const int* status, int* host_status,
                               hipStream_t st) {
  const PanelUnits u(m * r, n, r);
  hipLaunchKernelGGL(store_panels_kernel, dim3(u.wgs), dim3(256), 0, st, A, m, B, n, r, rp, W, H,
                     u.rows, u.tiles, u.all, status, host_status);
  return hipGetLastError();
}

hipError_t launch_reset(float* a, int64_t na, float* b, int64_t nb, int* status, hipStream_t st) {
  const int64_t most = ((na > nb ? na : nb) / 4 + 255) / 256;
  const unsigned wgs = (unsigned)(most < 1 ? 1 : (most < 4096 ? most : 4096));
  hipLaunchKernelGGL(reset_kernel, dim3(wgs), dim3(256), 0, st, reinterpret_cast<float4*>(a), na / 4,
                     reinterpret_cast<float4*>(b), nb / 4, status);
  return hipGetLastError();
}

hipError_t launch_zero(float* p, int64_t count, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_kernel, dim3(blocks(count)), dim3(256), 0, st, p, count);
  return hipGetLastError();
}

hipError_t launch_guarded_copy(const float* src, float* dst, int64_t count, const int* status,
                               hipStream_t st) {
  const int64_t n4 = count / 4;
  if (n4 > 0 && ((uintptr_t)src % 16 == 0) && ((uintptr_t)dst % 16 == 0)) {
    hipLaunchKernelGGL(guarded_copy_kernel, dim3(blocks(n4)), dim3(256), 0, st,
                       (const float4*)src, (float4*)dst, n4, status);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (count > 4 * n4)
      hipLaunchKernelGGL(guarded_copy_tail_kernel, dim3(1), dim3(256), 0, st, src, dst, 4 * n4,
                         count, status);
    return hipGetLastError();
  }
  if (count > 0)
    hipLaunchKernelGGL(guarded_copy_tail_kernel, dim3(blocks(count)), dim3(256), 0, st, src, dst,
                       (int64_t)0, count, status);
  return hipGetLastError();
}

hipError_t launch_guard(const double* q_old, const double* q_new, double tol2, int* status,
                        int step_id, hipStream_t st) {
  hipLaunchKernelGGL(guard_kernel, dim3(1), dim3(64), 0, st, q_old, q_new, tol2, status, step_id);
  return hipGetLastError();
}

hipError_t launch_sum(const double* partial, int64_t count, int n, double* out, int* is_nan,
                      const int* when, hipStream_t st) {
  hipLaunchKernelGGL(sum_kernel, dim3((unsigned)n), dim3(1024), 0, st, partial, count, out, is_nan,
                     when);
  return hipGetLastError();
}

}  // namespace nmd
