// Small utility kernels: max |x| over an array (facet sizing) and fills.
// Fills are kernels rather than hipMemsetAsync so that a captured graph
// holds only kernel nodes.
#include "rlf_devmath.h"
#include "rlf_internal.h"

namespace rlf {

namespace {

// out2[k] = max |x_k| of two arrays (blockIdx.y).  Few blocks, each with
// eight loads of a thread in flight: 1,158,361 values of both arrays take
// 12 us; with a block per 256 values the thousands of atomics on one
// address took 109.
constexpr int kAbsmaxBlocks = 256;

__global__ __launch_bounds__(256) void k_absmax(const double *x, const double *y, int64_t n, double *out2) {
  __shared__ double sh[4];
  const double *p = blockIdx.y ? y : x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  double m = 0.0;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i + 7 * stride < n; i += 8 * stride) {
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = p[i + k * stride];
#pragma unroll
    for (int k = 0; k < 8; ++k) m = fmax(m, fabs(v[k]));
  }
  for (; i < n; i += stride) m = fmax(m, fabs(p[i]));
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) m = fmax(m, __shfl_xor(m, d));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    // non-negative doubles order like their bit patterns
    atomicMax(reinterpret_cast<unsigned long long *>(out2 + blockIdx.y), (unsigned long long)__double_as_longlong(m));
  }
}

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t *p, int64_t n, uint32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

__global__ __launch_bounds__(256) void k_fill_cis(double2 *master) { cis_table_init<kCisMaster>(master); }

// dst[idx[i]] = src[i] (| bits for the 32-bit form), i < n; idx in range by
// construction of the caller.
__global__ __launch_bounds__(256) void k_scatter_f64(const double *src, const int32_t *idx, int64_t n, double *dst) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    dst[idx[i]] = src[i];
}

__global__ __launch_bounds__(256) void k_scatter_u32(const uint32_t *src, const int32_t *idx, int64_t n, uint32_t bits,
                                                     uint32_t *dst) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    dst[idx[i]] = src[i] | bits;
}

// One job per blockIdx.y, 16 bytes per access where both ends allow it.  A
// copy command for each of fourteen small tables cost the host and the stream
// 10 us apiece; this launch replaces them.
__global__ __launch_bounds__(256) void k_copy_jobs(CopyJobs j) {
  const auto &job = j.job[blockIdx.y];
  const size_t first = (size_t)blockIdx.x * 256 + threadIdx.x, stride = (size_t)gridDim.x * 256;
  size_t done = 0;
  if (((reinterpret_cast<uintptr_t>(job.dst) | reinterpret_cast<uintptr_t>(job.src)) & 15) == 0) {
    const size_t n = job.bytes / 16;
    const uint4 *src = static_cast<const uint4 *>(job.src);
    uint4 *dst = static_cast<uint4 *>(job.dst);
    for (size_t i = first; i < n; i += stride) dst[i] = src ? src[i] : make_uint4(0, 0, 0, 0);
    done = n * 4;
  }
  const uint32_t *src = static_cast<const uint32_t *>(job.src);
  uint32_t *dst = static_cast<uint32_t *>(job.dst);
  for (size_t i = done + first; i < job.bytes / 4; i += stride) dst[i] = src ? src[i] : 0u;
}

unsigned grid_for(int64_t n) {
  const int64_t b = (n + 255) / 256;
  return (unsigned)(b < 8192 ? (b > 0 ? b : 1) : 8192);
}

}  // namespace

hipError_t launch_absmax(const double *x, const double *y, int64_t n, double *out2, hipStream_t st) {
  const unsigned blocks = grid_for(n) < kAbsmaxBlocks ? grid_for(n) : kAbsmaxBlocks;
  hipLaunchKernelGGL(k_absmax, dim3(blocks, 2), dim3(256), 0, st, x, y, n, out2);
  return hipGetLastError();
}

hipError_t launch_scatter_f64(const double *src, const int32_t *idx, int64_t n, double *dst, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter_f64, dim3(grid_for(n)), dim3(256), 0, st, src, idx, n, dst);
  return hipGetLastError();
}

hipError_t launch_scatter_u32(const uint32_t *src, const int32_t *idx, int64_t n, uint32_t bits, uint32_t *dst,
                              hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter_u32, dim3(grid_for(n)), dim3(256), 0, st, src, idx, n, bits, dst);
  return hipGetLastError();
}

hipError_t launch_copy_jobs(const CopyJobs &j, hipStream_t st) {
  if (j.n <= 0) return hipSuccess;
  size_t most = 0;
  for (int k = 0; k < j.n; ++k) most = j.job[k].bytes > most ? j.job[k].bytes : most;
  const unsigned blocks = (unsigned)((most + 4095) / 4096 < 256 ? (most + 4095) / 4096 : 256);
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy_jobs, dim3(blocks, (unsigned)j.n), dim3(256), 0, st, j);
  return hipGetLastError();
}

hipError_t launch_fill_cis(double2 *master, hipStream_t st) {
  hipLaunchKernelGGL(k_fill_cis, dim3(1), dim3(256), 0, st, master);
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(n)), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

}  // namespace rlf
