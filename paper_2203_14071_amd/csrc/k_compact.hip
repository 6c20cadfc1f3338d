// Facet compaction (Sec. 2.3): keep the cells of each source's dense block
// that received at least one visibility, in memory order of the block, which
// is (iy, ix) order.  Vbar = Z / W; the cell centre is (ix, iy) / theta.  The
// FP64 likelihood's records are written folded (a cell and its mirror image
// as one).
// Three steps: count per source, scan over sources (in the write step of
// catalogues up to kOwnScan sources), write; the write step also clears the
// dense block for the next extraction.
#include "rlf_internal.h"

namespace rlf {

namespace {

__device__ __forceinline__ int block_sum_int(int x, int *sh) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) x += __shfl_xor(x, d);
  if (lane == 0) sh[wid] = x;
  __syncthreads();
  int t = 0;
  for (int k = 0; k < (int)(blockDim.x >> 6); ++k) t += sh[k];
  __syncthreads();
  return t;
}

// Cells of each source, and folded cells (a cell and its mirror image, flat
// indices k and n - 1 - k of the dense block, counted once).
__global__ __launch_bounds__(256) void k_count(CompactArgs a) {
  __shared__ int sh[4];
  const int s = blockIdx.x;
  const SrcGeom g = a.geom[s];
  const int64_t n = (int64_t)g.side * g.side;      // odd: the middle cell is its own mirror image
  const double4 *cell = a.acc.cell + g.base;
  int local = 0, folded = 0;
  for (int64_t k = threadIdx.x; k <= n / 2; k += blockDim.x) {
    const bool own = cell[k].w > 0.0, mirror = cell[n - 1 - k].w > 0.0;
    local += (int)own + (int)(mirror && k < n / 2);
    folded += own || mirror;
  }
  const int t = block_sum_int(local, sh), tf = block_sum_int(folded, sh);
  if (threadIdx.x == 0) {
    a.cells.n_nonempty[s] = t;
    a.cells.n_fold[s] = tf;
  }
}

// Up to this many sources each block of k_write adds up the counts of the
// sources before its own, of both kinds, eight loads per thread at most: k_write takes
// 5 us for 10 sources and 37 for 1,000 either way, and k_scan's 4.5 us are saved.
constexpr int kOwnScan = 1024;

// Exclusive scans over sources (block 0: cells, block 1: folded cells).
__global__ __launch_bounds__(1024) void k_scan(CompactArgs a) {
  __shared__ int64_t sh[1024];
  const int64_t *cnt = blockIdx.x == 0 ? a.cells.n_nonempty : a.cells.n_fold;
  int64_t *off = blockIdx.x == 0 ? a.cells.offsets : a.cells.fold_offsets;
  const int n = a.n_src;
  const int per = (n + 1023) / 1024;
  const int lo = min(n, (int)threadIdx.x * per), hi = min(n, lo + per);
  int64_t local = 0;
  for (int k = lo; k < hi; ++k) local += cnt[k];
  sh[threadIdx.x] = local;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {               // Hillis-Steele inclusive scan
    const int64_t o = threadIdx.x >= (unsigned)d ? sh[threadIdx.x - d] : 0;
    __syncthreads();
    sh[threadIdx.x] += o;
    __syncthreads();
  }
  int64_t run = sh[threadIdx.x] - local;
  for (int k = lo; k < hi; ++k) {
    off[k] = run;
    run += cnt[k];
  }
  if (threadIdx.x == 1023) off[n] = sh[1023];
}

// Position of this thread's item among the block's kept ones, and their number.
__device__ __forceinline__ int block_rank(bool keep, int *wsum, int &total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint64_t m = __ballot(keep);
  const int before = __popcll(m & ((1ull << lane) - 1ull));
  if (lane == 0) wsum[wid] = __popcll(m);
  __syncthreads();
  int wave_off = 0;
  total = 0;
  for (int q = 0; q < 4; ++q) {
    wave_off += q < wid ? wsum[q] : 0;
    total += wsum[q];
  }
  __syncthreads();
  return wave_off + before;
}

// Likelihood record with sqrt(W) carried by the profile: with c = W^{-1/3},
// sqrt(W) f(x) = (c x)^{-3/2} and c x = c + s_k |A^{-T} k'|^2 for the cell
// centre k' = W^{-1/6} (uc, vc), so a knot's terms are h = (c + s_k q')^{-3/2},
// D += (sqrt(W) Re Vbar) h, M += h h.
__device__ __forceinline__ double4 fit_record(int ix, int iy, double theta, double W, double vr) {
  const double uc = (double)ix / theta, vc = (double)iy / theta;
  const double cw = 1.0 / cbrt(W), rw = sqrt(cw);
  return make_double4(uc * rw, vc * rw, cw, sqrt(W) * vr);
}

// Cells in memory order of the dense block, and the folded records of the
// FP64 likelihood: f is even in (u, v), so the terms of a cell and of its
// mirror image, W Re(Vbar) f and W f^2, add before f is known.  An aperture-
// synthesis track covers both halves of the plane, so this nearly halves the
// likelihood's work: on the 197-antenna array 270 cells become 153 records
// per source, and extraction plus grid of 1000 sources take 22.7 ms (with
// the cells one by one 29.2; 300 sources, lattice-seeded, 1.26 and 2.01; 100
// sources over 5 x 5 offsets with the refinement 7.3 and 11.7).  The mixed
// form's grid keeps one FP32 record per cell (its results are those of the
// cells one by one); its FP64 recheck reads the folded ones.
template <bool kMixed>
__global__ __launch_bounds__(256) void k_write(CompactArgs a, int own_scan) {
  __shared__ int wsum[4];
  __shared__ int64_t osum[2][4];
  const int s = blockIdx.x;
  const SrcGeom g = a.geom[s];
  const double theta = a.src[s].theta;
  const int64_t n = (int64_t)g.side * g.side;
  int64_t out, fout;
  if (own_scan) {
    int64_t x = 0, f = 0;
    for (int k = threadIdx.x; k < s; k += blockDim.x) {
      x += a.cells.n_nonempty[k];
      f += a.cells.n_fold[k];
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      x += __shfl_xor(x, d);
      f += __shfl_xor(f, d);
    }
    if ((threadIdx.x & 63) == 0) {
      osum[0][threadIdx.x >> 6] = x;
      osum[1][threadIdx.x >> 6] = f;
    }
    __syncthreads();
    out = (osum[0][0] + osum[0][1]) + (osum[0][2] + osum[0][3]);
    fout = (osum[1][0] + osum[1][1]) + (osum[1][2] + osum[1][3]);
    if (threadIdx.x == 0) {
      a.cells.offsets[s] = out;
      a.cells.fold_offsets[s] = fout;
      if (s == a.n_src - 1) {
        a.cells.offsets[s + 1] = out + a.cells.n_nonempty[s];
        a.cells.fold_offsets[s + 1] = fout + a.cells.n_fold[s];
      }
    }
  } else {
    out = a.cells.offsets[s];
    fout = a.cells.fold_offsets[s];
  }
  for (int64_t k0 = 0; k0 < n; k0 += blockDim.x) {
    const int64_t k = k0 + threadIdx.x;
    double4 c = make_double4(0.0, 0.0, 0.0, 0.0), d = c;
    if (k < n) {
      c = a.acc.cell[g.base + k];
      if (k < n / 2) d = a.acc.cell[g.base + (n - 1 - k)];
    }
    const uint32_t cnt = (uint32_t)c.w;              // an exact integer sum
    const bool keep = cnt > 0u, fold = k <= n / 2 && (keep || d.w > 0.0);
    int total, ftotal;
    const int64_t o = out + block_rank(keep, wsum, total);
    const int64_t fo = fout + block_rank(fold, wsum, ftotal);
    // every read of this chunk is done (the ranks synchronise the block), and
    // a mirror cell still to be visited is cleared only then
    const int ix = (int)(k % g.side) - g.half;
    const int iy = (int)(k / g.side) - g.half;
    if (keep) {
      a.acc.cell[g.base + k] = make_double4(0.0, 0.0, 0.0, 0.0);
      const double vr = c.y / c.x, vi = c.z / c.x;
      a.cells.ix[o] = ix;
      a.cells.iy[o] = iy;
      a.cells.count[o] = (int32_t)cnt;
      a.cells.wsum[o] = c.x;
      a.cells.vre[o] = vr;
      a.cells.vim[o] = vi;
      if (kMixed) {
        const double4 r = fit_record(ix, iy, theta, c.x, vr);
        a.cells.fit32[o] = make_float4((float)r.x, (float)r.y, (float)r.z, (float)r.w);
      }
    }
    if (fold) {
      const double W = c.x + d.x;
      a.cells.fit64[fo] = fit_record(ix, iy, theta, W, (c.y + d.y) / W);
      if (!kMixed) a.cells.fold_aux[fo] = FoldAux{ix, iy, sqrt(W) * ((c.z - d.z) / W)};
    }
    out += total;
    fout += ftotal;
  }
}

}  // namespace

hipError_t launch_compact(const CompactArgs &a, int mixed, hipStream_t st) {
  hipLaunchKernelGGL(k_count, dim3(a.n_src), dim3(256), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int own_scan = a.n_src <= kOwnScan;
  if (!own_scan) {
    hipLaunchKernelGGL(k_scan, dim3(2), dim3(1024), 0, st, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (mixed)
    hipLaunchKernelGGL(k_write<true>, dim3(a.n_src), dim3(256), 0, st, a, own_scan);
  else
    hipLaunchKernelGGL(k_write<false>, dim3(a.n_src), dim3(256), 0, st, a, own_scan);
  return hipGetLastError();
}

}  // namespace rlf
