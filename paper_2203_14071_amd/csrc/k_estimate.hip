// Shape estimate (Sec. 2.4, 4.1): per source, the maximum of ln L(e) over
// the evaluated grid points (smallest flat index on ties), the set
// {ln L >= ln Lmax + ln frac}, its likelihood-weighted mean and population
// covariance (weights exp(ln L - ln Lmax)), and the flags: bad variance,
// empty facet, maximum on an edge of the evaluated region.  One block per
// source; three passes over the source's grid values with block reductions.
//
// The set is cut at a threshold and the maximum is a comparison, so the
// estimate is discontinuous in ln L: a point within the arithmetic error of
// the threshold can go either way.  In the mixed form (ln L summed in FP32,
// error bounded by delta) every point within 2 delta of the threshold or
// below the maximum is evaluated again in FP64 first, so both decisions are
// those of FP64 arithmetic on the same facet; the weights of the other
// points keep their FP32-summed values.
#include "rlf_devmath.h"
#include "rlf_internal.h"

namespace rlf {

namespace {

// One block per source; the launch is bound by the latency of its chain of
// loads, reductions and barriers.  The block holds up to kHeld grid values in
// registers between its passes (the 81 x 81 grid has 6,333 points; larger
// grids are read again by every pass), lists the points of the set for the
// passes over them, and reduces the sums of a pass together: one source takes
// 10.5 us, against 20 with every pass reading the values and reducing sum by
// sum (1000 sources 28 us, against 45).  1,024 threads: 16 us (the held
// values spill); values held in LDS: 18 us.
// The mixed form's recheck is bound by its arithmetic, each candidate point
// taken by a whole wave: with the knots' logarithms and exponentials a
// lane each and the candidates dealt out evenly 1000 sources take 0.15 ms,
// against 0.29 with every lane forming all knots' and each wave its own
// neighbourhood's candidates.
constexpr int kThreads = 512, kWavesEst = kThreads / 64;
constexpr int kHeld = 14 * kThreads;
constexpr double kLnPowM32Scale = 0.40546510810816438198;   // ln(3/2)

// ln L(e) of source s at (e1, e2) in FP64, evaluated by one whole wave (all
// 64 lanes, uniform arguments): the lanes split the source's cells, knots in
// groups of four; per knot D and M are summed per lane and then across the
// wave, lane k forms the term of knot k, and ln L(e) = ln sum_k w_k
// L(e, alpha_k) as in the FP64 fit (the same terms, summed in another order).
// Every lane returns the same value.
__device__ double loglike_f64_wave(const EstimateArgs &a, int s, double e1, double e2) {
  const int lane = threadIdx.x & 63;
  const double det = 1.0 - e1 * e1 - e2 * e2;
  const double g = 1.0 / (det * det);
  const double a11 = 1.0 + e1, a12 = e2, a22 = 1.0 - e1;
  const int64_t c0 = a.fold_offsets[s], c1 = a.fold_offsets[s + 1];
  const double *lw = a.logw + (int64_t)s * a.num_r;
  double own_d = 0.0, own_m = 1.0;                 // the sums of knot `lane`
  for (int k0 = 0; k0 < a.num_r; k0 += 4) {
    double D[4], M[4], sk[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      D[k] = M[k] = 0.0;
      sk[k] = k0 + k < a.num_r ? a.sk[k0 + k] * g : 0.0;
    }
    for (int64_t c = c0 + lane; c < c1; c += 64) {
      const double4 cl = a.fit64[c];
      const double ku = fma(a11, cl.x, a12 * cl.y);
      const double kv = fma(a12, cl.x, a22 * cl.y);
      const double q = fma(ku, ku, kv * kv);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double h = pow_m32_f64(fma(sk[k], q, cl.z));        // (2/3) sqrt(W) f_c
        D[k] = fma(cl.w, h, D[k]);
        M[k] = fma(h, h, M[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
      for (int d = 32; d > 0; d >>= 1) {
        D[k] += __shfl_xor(D[k], d);
        M[k] += __shfl_xor(M[k], d);
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (lane == k0 + k) {
        own_d = D[k];
        own_m = M[k];
      }
  }
  static_assert(kMaxKnots <= 64, "a lane per knot");
  const bool knot = lane < a.num_r;
  // D and M carry (2/3) and (4/9) of their values: ln M is off by -2 ln(3/2)
  const double v =
      knot ? lw[lane] + (own_d * own_d / (2.0 * own_m) - 0.5 * log(own_m) - kLnPowM32Scale) : -INFINITY;
  double mx = v;
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) mx = fmax(mx, __shfl_xor(mx, d));
  double acc = knot ? exp(v - mx) : 0.0;
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) acc += __shfl_xor(acc, d);
  return mx + log(acc);
}

// Sums of N values over the block, in the order of the waves; sh holds
// N * kWavesEst values.
template <int N>
__device__ __forceinline__ void block_sum(double (&x)[N], double *sh) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < N; ++i) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) x[i] += __shfl_xor(x[i], d);
    if (lane == 0) sh[i * kWavesEst + wid] = x[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    x[i] = 0.0;
#pragma unroll
    for (int w = 0; w < kWavesEst; ++w) x[i] += sh[i * kWavesEst + w];
  }
  __syncthreads();
}

__device__ __forceinline__ bool grid_valid(int i1, int i2, int n_e, int r2) {
  const int c = (n_e - 1) / 2;
  if (i1 < 0 || i2 < 0 || i1 >= n_e || i2 >= n_e) return false;
  return (i1 - c) * (i1 - c) + (i2 - c) * (i2 - c) < r2;
}

__device__ __forceinline__ bool in_box(const int32_t *win, int s, int i1, int i2) {
  if (!win) return true;
  const int4 b = reinterpret_cast<const int4 *>(win)[s];
  return i1 >= b.x && i1 <= b.y && i2 >= b.z && i2 <= b.w;
}

template <bool kRecheck>
__global__ __launch_bounds__(kThreads) void k_estimate(EstimateArgs a) {
  __shared__ double shd[4 * kWavesEst];
  __shared__ double shv[kWavesEst];
  __shared__ int shi[kWavesEst];
  __shared__ int touch;
  __shared__ uint16_t list[kHeld];
  const int s = blockIdx.x;
  if (a.redo && !a.redo[s]) return;
  double *L = a.lsurf + (int64_t)s * a.n_valid;
  const int64_t n_cells = a.offsets[s + 1] - a.offsets[s];
  const uint32_t extra = a.redo ? (uint32_t)RLF_FLAG_FALLBACK : 0u;
  const int ctr = (a.n_e - 1) / 2;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;

  // fn(j, ln L) for this thread's points, increasing j
  constexpr int kPer = kHeld / kThreads;
  double held[kPer];
  const bool hold = a.n_valid <= kHeld;
  auto fill = [&]() {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int j = (int)threadIdx.x + i * kThreads;
      held[i] = hold && n_cells > 0 && j < a.n_valid ? L[j] : 0.0;
    }
  };
  auto each = [&](auto &&fn) {
    if (hold) {
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const int j = (int)threadIdx.x + i * kThreads;
        if (j < a.n_valid) fn(j, held[i]);
      }
    } else {
      for (int j = threadIdx.x; j < a.n_valid; j += kThreads) fn(j, L[j]);
    }
  };
  fill();
  // where this thread's n entries go in a list over the block, and its length
  auto wave_base = [&](int n, int &at, int &total) {
    int x = n;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int o = __shfl_up(x, d);
      x += lane >= d ? o : 0;
    }
    if (lane == 63) shi[wid] = x;
    __syncthreads();
    at = x - n;
    total = 0;
    for (int q = 0; q < kWavesEst; ++q) {
      at += q < wid ? shi[q] : 0;
      total += shi[q];
    }
    __syncthreads();
  };

  // pass 1: maximum, smallest index on ties (each thread scans increasing j)
  double best;
  int bi;
  auto find_max = [&]() {
    best = -INFINITY;
    bi = 0x7fffffff;
    if (n_cells > 0) {
      each([&](int j, double v) {
        if (a.window) {
          const int f = a.epts[j];
          const int i1 = f / a.n_e, i2 = f - i1 * a.n_e;
          if (!in_box(a.window, s, i1, i2)) return;
        }
        if (v > best) {
          best = v;
          bi = j;
        }
      });
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      const double ov = __shfl_xor(best, d);
      const int oi = __shfl_xor(bi, d);
      if (ov > best || (ov == best && oi < bi)) {
        best = ov;
        bi = oi;
      }
    }
    if (lane == 0) {
      shv[wid] = best;
      shi[wid] = bi;
    }
    __syncthreads();
    best = shv[0];
    bi = shi[0];
    for (int q = 1; q < kWavesEst; ++q)
      if (shv[q] > best || (shv[q] == best && shi[q] < bi)) {
        best = shv[q];
        bi = shi[q];
      }
    __syncthreads();
  };
  find_max();

  // FP64 recheck (mixed form): the points that can decide the maximum or sit
  // at the threshold, each evaluated by a whole wave; the waves own disjoint
  // points, and every read of a point's FP32-summed value precedes its write
  if (kRecheck && best > -INFINITY) {
    const double delta = a.recheck_rel * (fabs(best) + a.recheck_abs);
    const double lo = best - 2.0 * delta, thr0 = best + a.log_frac;
    const bool lat_out = a.redo_out && a.check_stride > 0;
    auto candidate = [&](int j, double v) {
      const int f = a.epts[j];
      const int i1 = f / a.n_e, i2 = f - i1 * a.n_e;
      if (in_box(a.window, s, i1, i2)) return v >= lo || fabs(v - thr0) <= 2.0 * delta;
      return lat_out && (i1 - ctr) % a.check_stride == 0 && (i2 - ctr) % a.check_stride == 0 &&
             fabs(v - thr0) <= 2.0 * delta;
    };
    auto evaluate = [&](int j) {                   // by the whole wave
      const int f = a.epts[j];
      const int i1 = f / a.n_e, i2 = f - i1 * a.n_e;
      const double v = loglike_f64_wave(a, s, (double)(i1 - ctr) * a.e_step, (double)(i2 - ctr) * a.e_step);
      if (lane == 0) L[j] = v;
    };
    if (hold) {
      // the candidates are neighbours on the grid: dealt out to the waves from
      // a list, so that none has most of them
      uint32_t mine = 0;                           // bit i: held[i] is one
#pragma unroll 1
      for (int i = 0; i < kPer; ++i) {
        const int j = (int)threadIdx.x + i * kThreads;
        if (j < a.n_valid && candidate(j, L[j])) mine |= 1u << i;
      }
      int at, n_cand;
      wave_base(__popc(mine), at, n_cand);
      for (; mine; mine &= mine - 1) list[at++] = (uint16_t)((int)threadIdx.x + (__ffs(mine) - 1) * kThreads);
      __syncthreads();
      for (int t = wid; t < n_cand; t += kWavesEst) evaluate(list[t]);
    } else {
      for (int j0 = wid * 64; j0 < a.n_valid; j0 += kThreads) {
        const int j = j0 + lane;
        uint64_t m = __ballot(j < a.n_valid && candidate(j, L[j]));
        for (; m; m &= m - 1) evaluate(j0 + __ffsll((unsigned long long)m) - 1);
      }
    }
    __threadfence_block();
    __syncthreads();
    fill();
    find_max();
  }

  if (a.surface) {
    double *S = a.surface + (int64_t)s * a.n_e * a.n_e;
    for (int f = threadIdx.x; f < a.n_e * a.n_e; f += kThreads) {
      const int i1 = f / a.n_e, i2 = f - i1 * a.n_e;
      if (!grid_valid(i1, i2, a.n_e, a.half_r2)) S[f] = -INFINITY;
    }
    for (int j = threadIdx.x; j < a.n_valid; j += kThreads) {
      const int f = a.epts[j];
      const int i1 = f / a.n_e, i2 = f - i1 * a.n_e;
      S[f] = (n_cells > 0 && in_box(a.window, s, i1, i2)) ? L[j] : -INFINITY;
    }
  }

  if (!(best > -INFINITY)) {                   // empty facet or nothing evaluated
    if (threadIdx.x == 0) {
      const double nan = NAN;
      if (a.e1) a.e1[s] = nan;
      if (a.e2) a.e2[s] = nan;
      if (a.s1) a.s1[s] = nan;
      if (a.s2) a.s2[s] = nan;
      if (a.c12) a.c12[s] = nan;
      if (a.lmax) a.lmax[s] = nan;
      if (a.argmax) a.argmax[s] = -1;
      if (a.n_above) a.n_above[s] = 0;
      a.flags[s] = (uint32_t)RLF_FLAG_EMPTY | extra;
      // a window holding no valid grid point of a non-empty facet is refitted
      if (a.redo_out) a.redo_out[s] = n_cells > 0 ? 1 : 0;
    }
    return;
  }

  // pass 2: weight, first moments, count over the thresholded set; with a
  // window, also whether any member has a grid neighbour outside the window
  // (the set may continue beyond it: the narrowed result is not trusted) or
  // an evaluated lattice point outside the window reaches the set
  const double thr = best + a.log_frac;
  // the points of the set, in a list: the passes over them are short loops
  // over all threads
  int n_set = 0;
  if (hold) {
    uint32_t mine = 0;                             // bit i: held[i] is in the set
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if ((int)threadIdx.x + i * kThreads < a.n_valid && held[i] >= thr) mine |= 1u << i;
    int at;
    wave_base(__popc(mine), at, n_set);
    for (; mine; mine &= mine - 1) list[at++] = (uint16_t)((int)threadIdx.x + (__ffs(mine) - 1) * kThreads);
  }
  auto members = [&](auto &&fn) {
    if (hold) {
      for (int t = threadIdx.x; t < n_set; t += kThreads) fn((int)list[t], L[list[t]]);
    } else {
      for (int j = threadIdx.x; j < a.n_valid; j += kThreads)
        if (L[j] >= thr) fn(j, L[j]);
    }
  };
  double sum[4] = {0.0, 0.0, 0.0, 0.0};          // weight, first moments, count
  if (threadIdx.x == 0) touch = 0;
  __syncthreads();
  members([&](int j, double v) {
    const int f = a.epts[j];
    const int i1 = f / a.n_e, i2 = f - i1 * a.n_e;
    if (!in_box(a.window, s, i1, i2)) {
      // a lattice point outside the window reaching the set: refit
      if (a.redo_out && a.check_stride > 0 && (i1 - ctr) % a.check_stride == 0 &&
          (i2 - ctr) % a.check_stride == 0)
        atomicOr(&touch, 1);
      return;
    }
    if (a.window && a.redo_out) {
      const int nb[4][2] = {{1, 0}, {-1, 0}, {0, 1}, {0, -1}};
      for (int q = 0; q < 4; ++q) {
        const int j1 = i1 + nb[q][0], j2 = i2 + nb[q][1];
        if (grid_valid(j1, j2, a.n_e, a.half_r2) && !in_box(a.window, s, j1, j2)) atomicOr(&touch, 1);
      }
    }
    const double w = exp(v - best);
    const double x1 = (double)(i1 - ctr) * a.e_step, x2 = (double)(i2 - ctr) * a.e_step;
    sum[0] += w;
    sum[1] += w * x1;
    sum[2] += w * x2;
    sum[3] += 1.0;
  });
  block_sum(sum, shd);
  const double sw = sum[0], cnt = sum[3];
  const double m1 = sum[1] / sw, m2 = sum[2] / sw;

  // pass 3: central second moments
  double sec[3] = {0.0, 0.0, 0.0};
  members([&](int j, double v) {
    const int f = a.epts[j];
    const int i1 = f / a.n_e, i2 = f - i1 * a.n_e;
    if (!in_box(a.window, s, i1, i2)) return;
    const double w = exp(v - best);
    const double d1 = (double)(i1 - ctr) * a.e_step - m1, d2 = (double)(i2 - ctr) * a.e_step - m2;
    sec[0] += w * d1 * d1;
    sec[1] += w * d2 * d2;
    sec[2] += w * d1 * d2;
  });
  block_sum(sec, shd);
  const double c11 = sec[0] / sw, c22 = sec[1] / sw, c12 = sec[2] / sw;

  if (threadIdx.x == 0) {
    const double sd1 = sqrt(c11), sd2 = sqrt(c22);
    const double det = c11 * c22 - c12 * c12;
    const double sqd = det > 0.0 ? sqrt(det) : 0.0;
    uint32_t fl = extra;
    if (sd1 <= a.bad_sigma || sd2 <= a.bad_sigma || sqd <= a.bad_sqrtdet) fl |= RLF_FLAG_BAD_VAR;
    const int f = a.epts[bi];
    const int i1 = f / a.n_e, i2 = f - i1 * a.n_e;
    bool edge = i1 == 0 || i2 == 0 || i1 == a.n_e - 1 || i2 == a.n_e - 1;
    bool inner_edge = false;
    const int nb[4][2] = {{1, 0}, {-1, 0}, {0, 1}, {0, -1}};
    for (int q = 0; q < 4; ++q) {
      const int j1 = i1 + nb[q][0], j2 = i2 + nb[q][1];
      const bool gv = grid_valid(j1, j2, a.n_e, a.half_r2);
      const bool inw = in_box(a.window, s, j1, j2);
      if (!(gv && inw)) edge = true;
      if (gv && !inw) inner_edge = true;
    }
    if (edge) fl |= RLF_FLAG_EDGE;
    if (a.e1) a.e1[s] = m1;
    if (a.e2) a.e2[s] = m2;
    if (a.s1) a.s1[s] = sd1;
    if (a.s2) a.s2[s] = sd2;
    if (a.c12) a.c12[s] = c12;
    if (a.lmax) a.lmax[s] = best;
    if (a.argmax) a.argmax[s] = f;
    if (a.n_above) a.n_above[s] = (int32_t)cnt;
    a.flags[s] = fl;
    if (a.redo_out) a.redo_out[s] = (inner_edge || touch) ? 1 : 0;
  }
}

}  // namespace

hipError_t launch_estimate(const EstimateArgs &a, hipStream_t st) {
  if (a.fit64)
    hipLaunchKernelGGL(k_estimate<true>, dim3(a.n_src), dim3(kThreads), 0, st, a);
  else
    hipLaunchKernelGGL(k_estimate<false>, dim3(a.n_src), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace rlf
