// Likelihood grid (Sec. 2.4): for each source, ellipticity grid point e and
// scale-length knot alpha_k,
//   f_c = (1 + s_k q_c(e))^{-3/2},  q_c(e) = |A_e^{-T} k_c|^2,  s_k = 4 pi^2 alpha_k^2,
//   D_k = sum_c W_c f_c Re Vbar_c,  M_k = sum_c W_c f_c^2,
//   ln L(e, alpha_k) = D_k^2 / (2 M_k) - ln(M_k) / 2            (flux marginalised)
//   ln L(e) = m + ln sum_k exp(ln w_k + ln L(e, alpha_k) - m)   (scale marginalised)
//
// f is even in (u, v): in the FP64 form a cell and its mirror image are one
// record (W and W Re Vbar added, k_compact.hip), in the mixed form a record
// is one cell.
//
// One thread per grid point, all knots of that point in registers (D_k, M_k),
// a uniform loop over the source's cells: each cell record comes in through
// one scalar load shared by the wave; it carries sqrt(W_c) in the profile's
// scale, (W^{-1/6} uc, W^{-1/6} vc, W^{-1/3}, sqrt(W) Re Vbar), so that
// h = (W^{-1/3} + s_k q')^{-3/2} = sqrt(W_c) f_c (q' the quadratic form of the
// scaled centre).  Per (cell, point) the quadratic form costs 6 ops and
// serves all knots; per (cell, point, knot): 1 FMA, x^(-3/2), 2 FMAs
// (D += b h, M += h h).
//   FP64 form:  x^(-3/2) as v_rsq_f64 cubed with a first-order correction
//               (5 ops, relative error < 3e-14), computed as (2/3) x^(-3/2).
//   Mixed form: FP32 cell data and arithmetic (v_rsq_f32 cubed), partial sums of
//               each block of kBlock cells folded into FP64 totals, so the
//               FP32 rounding error grows with kBlock, not with the cell count.
// The epilogue (logs, exps, log-sum-exp over knots) is FP64 in both forms.
//
// Position marginalisation (Sec. 2.4; n_pos offsets x_p on a square grid,
// uniform prior): D is formed per offset from the cross-correlation data
// G[c, p] = sqrt(W_c) Re(Vbar_c exp(-2 pi i k_c.x_p)) and M is shared,
//   ln L(e) = ln sum_k w_k (1/n_pos) sum_p exp(D_kp^2 / (2 M_k) - ln(M_k) / 2).
// The knots run in blocks of KB with the KB * n_pos sums of a block in
// registers; the n_pos values of a cell come in through scalar loads (one
// row of G per cell, G carrying sqrt(W_c) as the records do: the profile
// term h is sqrt(W_c) f_c), so a (cell, point, knot) costs the profile (6
// ops), M (1) and one FMA per offset, plus the quadratic form once per knot
// block.
#include "rlf_cellsums.h"
#include "rlf_devmath.h"
#include "rlf_internal.h"

namespace rlf {

namespace {

constexpr int kBlock = kCellBlock;
constexpr double kLnPowM32Scale = 0.40546510810816438198;   // ln(3/2)
// Full grids of at most this many groups of 64 points (48 sources on the 81 x
// 81 grid) share their knots between waves (k_fit_knots).  Grid and estimate,
// us, k_fit | k_fit_knots: 81 x 81 points, 1, 10, 48 and 100 sources FP64 66 |
// 35, 99 | 70, 239 | 231 and 433 | 467, mixed 97 | 54, 131 | 81, 221 | 224 and
// 399 | 422; 21 x 21 points, 100, 500 and 1000 sources 132 | 66, 236 | 174 and
// 359 | 338, mixed 157 | 68, 213 | 168 and 330 | 317; 11 x 11, 100 and 1000
// sources 129 | 61 and 196 | 124.
constexpr int64_t kKnotGroups = 48 * 99;

// Knots per pass over the cells: the mixed form with 20 knots takes them in
// two passes of 10 (the quadratic form is formed twice per cell, but half
// the accumulators leave room for twice the resident waves: measured 6 %
// faster); the FP64 form is faster in one pass.
template <int R, bool kMixed>
constexpr int knots_per_pass() { return (kMixed && R == 20) ? 10 : R; }

// A log-sum-exp in the making: ln of the terms so far = mx + ln(acc).
struct Lse {
  double mx = -INFINITY, acc = 0.0;
  // Add the n terms exp(v[k]).
  template <int N>
  __device__ __forceinline__ void add(const double (&v)[N], int n) {
    double bm = -INFINITY;
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (k < n) bm = fmax(bm, v[k]);
    const double nm = fmax(mx, bm);
    double bs = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (k < n) bs += exp(v[k] - nm);
    acc = (mx > -INFINITY ? acc * exp(mx - nm) : 0.0) + bs;
    mx = nm;
  }
};

// The terms ln(w_k L(e, alpha_k)) of source s (not empty) at (e1, e2),
// |e| < 1, for the n <= KP knots from k0 on: one pass over the source's
// records.
template <int KP, bool kMixed>
__device__ __forceinline__ void knot_terms(const FitArgs &a, int s, double e1, double e2, int k0, int n,
                                           double (&D)[KP]) {
  const double det = 1.0 - e1 * e1 - e2 * e2;
  const double g = 1.0 / (det * det);
  const int64_t c0 = a.offsets[s], c1 = a.offsets[s + 1];
  const double *lw = a.logw + (int64_t)s * a.num_r;
  double M[KP];
#pragma unroll
  for (int k = 0; k < KP; ++k) D[k] = M[k] = 0.0;
  if (!kMixed) {
    // A^{-T} with its 1/det folded in, so that the knot scales s_k stay
    // wave-uniform (SGPR operands: 40 VGPRs fewer than per-lane s_k g)
    const double id = 1.0 / det;
    const double a11 = (1.0 + e1) * id, a12 = e2 * id, a22 = (1.0 - e1) * id;
    double sk[KP];
#pragma unroll
    for (int k = 0; k < KP; ++k) sk[k] = k < n ? a.sk[k0 + k] : 0.0;
    cell_sums_f64<KP>(a.fit64, c0, c1, a11, a12, a22, sk, n, D, M);
  } else {
    const float a11 = (float)(1.0 + e1), a12 = (float)e2, a22 = (float)(1.0 - e1);
    float sk[KP];
#pragma unroll
    for (int k = 0; k < KP; ++k) sk[k] = k < n ? (float)(a.sk[k0 + k] * g) : 0.0f;
    cell_sums_f32<KP>(a.fit32, c0, c1, a11, a12, a22, sk, n, D, M);
  }
  // ln(w_k L(e, alpha_k)) in place of D; FP64 form: D and M carry (2/3)
  // and (4/9) of their values, so the ratio term is unchanged and ln M is
  // off by ln(4/9) = -2 ln(3/2)
#pragma unroll
  for (int k = 0; k < KP; ++k)
    if (k < n) D[k] = lw[k0 + k] + (D[k] * D[k] / (2.0 * M[k]) - 0.5 * log(M[k]) - (kMixed ? 0.0 : kLnPowM32Scale));
}

// ln L(e) of source s at (e1, e2), |e| < 1; NaN for an empty facet.
template <int R, bool kExact, bool kMixed>
__device__ __forceinline__ double loglike_e(const FitArgs &a, int num_r_arg, int s, double e1, double e2) {
  constexpr int KP = knots_per_pass<R, kMixed>();
  if (a.offsets[s + 1] == a.offsets[s]) return NAN;
  const int num_r = kExact ? R : num_r_arg;
  Lse t;
#pragma unroll 1
  for (int k0 = 0; k0 < R; k0 += KP) {
    if (k0 >= num_r) break;
    double v[KP];
    knot_terms<KP, kMixed>(a, s, e1, e2, k0, num_r - k0, v);
    t.add(v, num_r - k0);
  }
  return t.mx + log(t.acc);
}

// Knots per block of the position-marginalised sum: KB * NP partial sums
// in registers (FP64, plus as many FP32 ones in the mixed form).
constexpr int pos_knot_block(int np) { return np <= 9 ? 4 : (np <= 25 ? 2 : 1); }

// The position-marginalised terms, sum over the offsets included, of the
// blocks of KB = pos_knot_block(NP) knots from kfirst on in steps of kstep.
template <int NP, bool kMixed>
__device__ __forceinline__ void add_knots_pos(const FitArgs &a, int num_r, int s, double e1, double e2, int kfirst,
                                              int kstep, Lse &acc_out) {
  constexpr int KB = pos_knot_block(NP);
  const double det = 1.0 - e1 * e1 - e2 * e2;
  const double g = 1.0 / (det * det);
  const int64_t c0 = a.offsets[s], c1 = a.offsets[s + 1];
  const double *lw = a.logw + (int64_t)s * a.num_r;
  double mx = acc_out.mx, acc = acc_out.acc;
#pragma unroll 1
  for (int k0 = kfirst; k0 < num_r; k0 += kstep) {
    double D[KB][NP], M[KB];
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      M[b] = 0.0;
#pragma unroll
      for (int p = 0; p < NP; ++p) D[b][p] = 0.0;
    }
    if (!kMixed) {
      const double a11 = 1.0 + e1, a12 = e2, a22 = 1.0 - e1;
      double sk[KB];
#pragma unroll
      for (int b = 0; b < KB; ++b) sk[b] = k0 + b < num_r ? a.sk[k0 + b] * g : 0.0;
      const double4 *__restrict__ cells = a.fit64;
      const double *__restrict__ G = a.pos_g64;
      // A cell's row of G arrives in chunks of at most 13 values through two
      // buffers of scalar registers: once a chunk is there, the next one (of
      // this cell or the next) is issued, and the chunk's FMAs cover its way.
      // Scalar loads return in any order, so a wait is for all of them: left
      // to itself the compiler waited for a whole row, or for every eight
      // values, with nothing in flight behind them.
      // (A row of 9 is one chunk, behind four knots' arithmetic.)
      constexpr int kChunks = NP <= 13 ? 1 : (NP <= 26 ? 2 : 4), CH = (NP + kChunks - 1) / kChunks;
      double buf[2][CH];
      double4 nx;
      auto load = [&](int64_t c, int ch, double(&b)[CH]) {
#pragma unroll
        for (int i = 0; i < CH; ++i)
          if (ch * CH + i < NP) b[i] = G[c * NP + ch * CH + i];
      };
      auto cell = [&](int64_t c) {
        const double4 cl = nx;
        const double ku = fma(a11, cl.x, a12 * cl.y);
        const double kv = fma(a12, cl.x, a22 * cl.y);
        const double q = fma(ku, ku, kv * kv);
        double f[KB];
#pragma unroll
        for (int b = 0; b < KB; ++b) {
          f[b] = pow_m32_f64(fma(sk[b], q, cl.z));                  // (2/3) sqrt(W) f_c
          M[b] = fma(f[b], f[b], M[b]);
        }
#pragma unroll
        for (int ch = 0; ch < kChunks; ++ch) {
          double(&have)[CH] = buf[ch & 1];
          double(&next)[CH] = buf[(ch + 1) & 1];
#pragma unroll
          for (int i = 0; i < CH; ++i)
            if (kChunks > 1 && ch * CH + i < NP) asm("" : "+s"(have[i]));             // arrived
          __builtin_amdgcn_sched_barrier(0);
          if (ch + 1 < kChunks) {
            load(c, ch + 1, next);
          } else if (kChunks > 1) {
            const int64_t cn = min(c + 1, c1 - 1);
            nx = cells[cn];
            load(cn, 0, next);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int i = 0; i < CH; ++i)
              if (ch * CH + i < NP) D[b][ch * CH + i] = fma(f[b], have[i], D[b][ch * CH + i]);
        }
      };
      if constexpr (kChunks > 1) {
        nx = cells[c0];
        load(c0, 0, buf[0]);
      }
      for (int64_t c = c0; c < c1; ++c) {
        if constexpr (kChunks == 1) {
          nx = cells[c];
          load(c, 0, buf[0]);
        }
        cell(c);
      }
    } else {
      const float a11 = (float)(1.0 + e1), a12 = (float)e2, a22 = (float)(1.0 - e1);
      float sk[KB];
#pragma unroll
      for (int b = 0; b < KB; ++b) sk[b] = k0 + b < num_r ? (float)(a.sk[k0 + b] * g) : 0.0f;
      const float4 *__restrict__ cells = a.fit32;
      const float *__restrict__ G = a.pos_g32;
      auto block = [&](int64_t cb, int n) {
        float d[KB][NP], m[KB];
#pragma unroll
        for (int b = 0; b < KB; ++b) {
          m[b] = 0.0f;
#pragma unroll
          for (int p = 0; p < NP; ++p) d[b][p] = 0.0f;
        }
        for (int t = 0; t < n; ++t) {
          const float4 cl = cells[cb + t];
          const float ku = fmaf(a11, cl.x, a12 * cl.y);
          const float kv = fmaf(a12, cl.x, a22 * cl.y);
          const float q = fmaf(ku, ku, kv * kv);
          const float *gc = G + (cb + t) * NP;
#pragma unroll
          for (int b = 0; b < KB; ++b) {
            const float r = __builtin_amdgcn_rsqf(fmaf(sk[b], q, cl.z));
            const float f = r * r * r;                                // sqrt(W) f_c
            m[b] = fmaf(f, f, m[b]);
#pragma unroll
            for (int p = 0; p < NP; ++p) d[b][p] = fmaf(f, gc[p], d[b][p]);
          }
        }
#pragma unroll
        for (int b = 0; b < KB; ++b) {
          M[b] += (double)m[b];
#pragma unroll
          for (int p = 0; p < NP; ++p) D[b][p] += (double)d[b][p];
        }
      };
      int64_t cb = c0;
#pragma clang loop unroll(disable)
      for (; cb + kBlock <= c1; cb += kBlock) block(cb, kBlock);
      if (cb < c1) block(cb, (int)(c1 - cb));
    }
    // ln(w_k L(e, alpha_k, x_p)) in place of D, then one rescaling of the
    // running sum per block
    double bm = -INFINITY;
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      if (k0 + b < num_r) {
        const double base = lw[k0 + b] - 0.5 * log(M[b]) - (kMixed ? 0.0 : kLnPowM32Scale);
        const double h = 1.0 / (2.0 * M[b]);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          D[b][p] = fma(D[b][p] * D[b][p], h, base);
          bm = fmax(bm, D[b][p]);
        }
      }
    }
    const double nm = fmax(mx, bm);
    double bs = 0.0;
#pragma unroll
    for (int b = 0; b < KB; ++b)
      if (k0 + b < num_r) {
#pragma unroll
        for (int p = 0; p < NP; ++p) bs += exp(D[b][p] - nm);
      }
    acc = (mx > -INFINITY ? acc * exp(mx - nm) : 0.0) + bs;
    mx = nm;
  }
  acc_out.mx = mx;
  acc_out.acc = acc;
}

// ln L(e) at valid grid point j (index into the valid-point list) of source s.
template <int R, bool kExact, bool kMixed>
__device__ __forceinline__ void eval_point(const FitArgs &a, int num_r, int s, int j) {
  const int idx = a.epts[j];
  const int i1 = idx / a.n_e, i2 = idx - (idx / a.n_e) * a.n_e;
  const int ctr = (a.n_e - 1) / 2;
  a.lsurf[(int64_t)s * a.n_valid + j] =
      loglike_e<R, kExact, kMixed>(a, num_r, s, (double)(i1 - ctr) * a.e_step, (double)(i2 - ctr) * a.e_step);
}

// Knots shared by waves: all waves of a block work on the same 64 points of
// one source, each on every fourth block of knots.  Position fixed, the terms
// meet in LDS and are summed in loglike_e's order (ln L is the same to the
// bit); marginalised, wave 0 joins the waves' log-sum-exps in their order.  A source's 6,333
// points are ~100 such blocks, and a wave's walk over the cells is NW times
// shorter than with all knots in one thread, so that a launch of few sources,
// or its largest facet, does not leave the chip idle; the records' scalar
// loads are shared.  It costs the quadratic form once per block of knots
// (6 operations to 11 per knot), nothing for the position-marginalised sum,
// whose knots come in blocks anyway.  Four waves: a fifth shares its SIMD with
// another (5 x 5 offsets, 100 sources: 3.9 ms with five waves, 2.2 with four).
// The refinement, whose windows of a few hundred points used to be one or two
// blocks per source, gains most: 100 sources, three levels, 0.63 -> 0.41 ms
// position-fixed, 3.0 -> 1.65 ms over 5 x 5 offsets, 4.3 -> 2.3 ms over 7 x 7.
template <bool kMixed, int NP>
struct KnotSplit {
  static constexpr int kKnots = NP ? pos_knot_block(NP) : 5;
  static constexpr int kWaves = 4;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kWavesPerSimd = NP == 0 ? 5 : (kMixed ? 2 : 3);
};

// Waves per block of the refinement.  Its windows are a few blocks per source,
// so the largest facet's walk bounds a level; with position offsets a wave
// holds the sums of 4, 2 or 1 knots only and four waves walk the records two,
// three or five times.  Ten waves take 20 knots of 25 offsets in one walk (as
// many as the FP64 sums' registers leave room for; eight in the mixed form):
// three levels for 100 sources, four waves | these: 9 offsets 491 | 344 us, 25
// 853 | 514, 49 1,741 | 1,046, 25 in the mixed form 1,146 | 828.
template <bool kMixed, int NP>
constexpr int refine_waves() { return NP == 0 ? 4 : (kMixed ? 8 : 10); }
template <bool kMixed, int NP>
constexpr int refine_waves_per_simd() { return NP == 0 ? 5 : (kMixed ? 2 : 3); }

// Doubles of LDS loglike_block needs with W waves.
template <int NP, int W>
constexpr int block_doubles() { return NP ? 2 * 64 * W : kMaxKnots * 64; }

// ln L(e) of source s (not empty) at one point per lane, the same points in
// every wave of the block; the result is wave 0's.
template <bool kMixed, int NP, int W>
__device__ __forceinline__ double loglike_block(const FitArgs &a, int num_r, int s, double e1, double e2, double *sh) {
  constexpr int KP = KnotSplit<kMixed, NP>::kKnots;
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if constexpr (NP != 0) {
    Lse t;
    add_knots_pos<NP, kMixed>(a, num_r, s, e1, e2, wid * KP, W * KP, t);
    sh[wid * 64 + lane] = t.mx;
    sh[(W + wid) * 64 + lane] = t.acc;
    __syncthreads();
    double nm = t.mx, acc = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) nm = fmax(nm, sh[w * 64 + lane]);
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const double m = sh[w * 64 + lane];
      acc += m > -INFINITY ? sh[(W + w) * 64 + lane] * exp(m - nm) : 0.0;   // (a wave without knots)
    }
    return nm > -INFINITY ? nm + log(acc / (double)NP) : NAN;   // every term NaN: a cell of the facet is
  } else {
#pragma unroll 1
    for (int k0 = wid * KP; k0 < num_r; k0 += W * KP) {
      double v[KP];
      if (k0 + KP <= num_r)
        knot_terms<KP, kMixed>(a, s, e1, e2, k0, KP, v);
      else
        knot_terms<KP, kMixed>(a, s, e1, e2, k0, num_r - k0, v);
#pragma unroll
      for (int k = 0; k < KP; ++k)
        if (k0 + k < num_r) sh[(k0 + k) * 64 + lane] = v[k];
    }
    __syncthreads();
    // loglike_e adds its terms pass by pass (the mixed form takes 20 knots in
    // two): the maximum of the passes so far, then the pass's exponentials,
    // here each by the wave that has the knot (bits as in loglike_e, those two
    // passes apart: there a few points differ by a unit in the last place)
    const int per = kMixed && num_r == 20 ? 10 : num_r;
    double mx[2] = {-INFINITY, -INFINITY};
#pragma unroll 4
    for (int k = 0; k < num_r; ++k) mx[k >= per] = fmax(mx[k >= per], sh[k * 64 + lane]);
    mx[1] = fmax(mx[0], mx[1]);
    __syncthreads();
#pragma unroll 1
    for (int k0 = wid * KP; k0 < num_r; k0 += W * KP)
#pragma unroll
      for (int k = 0; k < KP; ++k)
        if (k0 + k < num_r) sh[(k0 + k) * 64 + lane] = exp(sh[(k0 + k) * 64 + lane] - (k0 + k < per ? mx[0] : mx[1]));
    __syncthreads();
    double L = 0.0;
    if (wid == 0) {
      double acc = 0.0, bs = 0.0;
      for (int k = 0; k < per; ++k) acc += sh[k * 64 + lane];
      if (per < num_r) {
        for (int k = per; k < num_r; ++k) bs += sh[k * 64 + lane];
        acc = acc * exp(mx[0] - mx[1]) + bs;
      }
      L = mx[1] + log(acc);
    }
    return L;
  }
}

// Refinement level: the points of the source's window at resolution
// e_step / 2^level, 64 per block, e = k * that step, |e| < 1 tested on the
// integers; -inf outside the domain.  blockIdx.y = source, the grid sized for
// the largest window (blocks past a source's window leave at once).
template <bool kMixed, int NP>
__global__ __launch_bounds__((64 * refine_waves<kMixed, NP>()), (refine_waves_per_simd<kMixed, NP>())) void k_refine_eval(
    FitArgs a, RefineArgs r, int num_r) {
  constexpr int W = refine_waves<kMixed, NP>();
  __shared__ double sh[block_doubles<NP, W>()];
  const int s = blockIdx.y;
  const int32_t *w = r.win + (int64_t)s * 5;
  if (!w[0]) return;                           // (empty facets are never active)
  const int n1 = w[3], n2 = w[4], np = n1 * n2;
  const int64_t lim = (int64_t)r.unit << r.level;
  const double res = a.e_step / (double)(1 << r.level);
  const int t = blockIdx.x * 64 + (int)(threadIdx.x & 63);
  if ((int)blockIdx.x * 64 >= np) return;      // uniform
  const int64_t k1 = w[1] + min(t, np - 1) / n2, k2 = w[2] + min(t, np - 1) % n2;
  const bool in = k1 * k1 + k2 * k2 < lim * lim;
  // a point outside the domain is evaluated at the centre and dropped
  const double L = loglike_block<kMixed, NP, W>(a, num_r, s, in ? (double)k1 * res : 0.0, in ? (double)k2 * res : 0.0, sh);
  if (threadIdx.x < 64 && t < np) r.lloc[(int64_t)s * r.max_side * r.max_side + t] = in ? L : -INFINITY;
}

// Grid launch: blockIdx.y = source (largest facets first when a.size_order
// is set: blocks are dispatched in index order, and the long blocks of the
// largest facets then do not trail the launch), one thread per valid grid
// point.
template <int R, bool kExact, bool kMixed>
__global__ __launch_bounds__(256) void k_fit(FitArgs a, int num_r) {
  const int s = a.size_order ? a.size_order[a.n_src - 1 - (int)blockIdx.y] : (int)blockIdx.y;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= a.n_valid) return;
  if (a.redo && !a.redo[s]) return;
  eval_point<R, kExact, kMixed>(a, num_r, s, j);
}

// The grid with the knots shared by waves, for launches of few sources: the
// full grid of a small catalogue, the full refit of the sources a narrowed
// fit was not trusted for (blocks of the others leave at once), and the
// position-marginalised grids (mixed form: of few sources).  blockIdx.y =
// source, largest facets first; one group of 64 points per block (in a loop
// over groups the stores of one would keep the next one's record loads from
// being scalar).
template <bool kMixed, int NP>
__global__ __launch_bounds__((KnotSplit<kMixed, NP>::kThreads), (KnotSplit<kMixed, NP>::kWavesPerSimd)) void k_fit_knots(
    FitArgs a, int num_r) {
  __shared__ double sh[block_doubles<NP, KnotSplit<kMixed, NP>::kWaves>()];
  const int s = a.size_order ? a.size_order[a.n_src - 1 - (int)blockIdx.y] : (int)blockIdx.y;
  if (a.redo && !a.redo[s]) return;            // uniform
  const int j = blockIdx.x * 64 + (int)(threadIdx.x & 63);
  const int idx = a.epts[min(j, a.n_valid - 1)];
  const int i1 = idx / a.n_e, i2 = idx - (idx / a.n_e) * a.n_e;
  const int ctr = (a.n_e - 1) / 2;
  double L = NAN;
  if (a.offsets[s + 1] != a.offsets[s])        // uniform
    L = loglike_block<kMixed, NP, KnotSplit<kMixed, NP>::kWaves>(a, num_r, s, (double)(i1 - ctr) * a.e_step, (double)(i2 - ctr) * a.e_step, sh);
  if (threadIdx.x < 64 && j < a.n_valid) a.lsurf[(int64_t)s * a.n_valid + j] = L;
}

// The position-marginalised grid with all knots in a thread, for launches of
// many sources in the mixed form: its sums (FP32 partial ones and FP64 totals)
// leave two waves per SIMD either way, so that sharing the knots adds waves
// only where there are few.  300 and 1000 sources, us, k_fit_knots | this: 3 x
// 3 offsets 4,186 | 3,148 and 14,252 | 10,635, 5 x 5 8,379 | 7,179 and 28,548
// | 24,210, 7 x 7 21,981 | 15,457 and 75,007 | 52,326.
template <int NP>
__global__ __launch_bounds__(256) void k_fit_pos(FitArgs a, int num_r) {
  const int s = a.size_order ? a.size_order[a.n_src - 1 - (int)blockIdx.y] : (int)blockIdx.y;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= a.n_valid) return;
  const int idx = a.epts[j];
  const int i1 = idx / a.n_e, i2 = idx - (idx / a.n_e) * a.n_e;
  const int ctr = (a.n_e - 1) / 2;
  double L = NAN;
  if (a.offsets[s + 1] != a.offsets[s]) {      // uniform
    Lse t;
    add_knots_pos<NP, true>(a, num_r, s, (double)(i1 - ctr) * a.e_step, (double)(i2 - ctr) * a.e_step, 0,
                            pos_knot_block(NP), t);
    L = t.mx + log(t.acc / (double)NP);
  }
  a.lsurf[(int64_t)s * a.n_valid + j] = L;
}

// The positions of a windowed launch of source s: its inclusive box (i1lo,
// i1hi, i2lo, i2hi) in row-major order, then, with a check stride S, the
// lattice points c + S q (both axes, |q| <= c / S) outside the box.  No other
// point is evaluated (the estimator reads no other).
struct Window {
  int4 b;                                     // the box's part on the grid: at most n_e^2 positions
  int w2, span, nl, ctr;
  bool by_valid;
  __device__ __forceinline__ Window(const FitArgs &a, int s) {
    // lattice pass 1: the lattice alone (an empty box); pass 2: the lattice
    // values are already in the surface, only the box is evaluated
    b = a.lattice_pass == 1 ? make_int4(1, 0, 1, 0) : reinterpret_cast<const int4 *>(a.window)[s];
    b.x = max(b.x, 0);
    b.y = min(b.y, a.n_e - 1);
    b.z = max(b.z, 0);
    b.w = min(b.w, a.n_e - 1);
    w2 = b.w >= b.z ? b.w - b.z + 1 : 1;
    const int area = (b.y >= b.x && b.w >= b.z) ? (b.y - b.x + 1) * w2 : 0;
    ctr = (a.n_e - 1) / 2;
    const int h = a.check_stride > 0 ? ctr / a.check_stride : 0;
    nl = (a.check_stride > 0 && a.lattice_pass != 2) ? 2 * h + 1 : 0;
    // a box with at least as many positions as the grid has valid points is
    // walked over the valid points instead (no idle lanes on |e| >= 1)
    by_valid = area >= a.n_valid;
    span = by_valid ? a.n_valid : area;
  }
  __device__ __forceinline__ int positions() const { return span + nl * nl; }
  // The valid point of position t, -1 for none: |e| >= 1, evaluated with the
  // box, or past the source's positions.
  __device__ __forceinline__ int point(const FitArgs &a, int t) const {
    if (t >= positions()) return -1;
    int i1, i2;
    if (by_valid && t < span) {
      const int f = a.epts[t];
      i1 = f / a.n_e;
      i2 = f - i1 * a.n_e;
      return i1 >= b.x && i1 <= b.y && i2 >= b.z && i2 <= b.w ? t : -1;
    }
    if (t < span) {
      i1 = b.x + t / w2;
      i2 = b.z + t % w2;
    } else {
      const int u = t - span, h = (nl - 1) / 2;
      i1 = ctr + a.check_stride * (u / nl - h);
      i2 = ctr + a.check_stride * (u % nl - h);
      if (i1 >= b.x && i1 <= b.y && i2 >= b.z && i2 <= b.w) return -1;
    }
    if (i1 < 0 || i2 < 0 || i1 >= a.n_e || i2 >= a.n_e) return -1;
    return a.valid_index[i1 * a.n_e + i2];
  }
};

// Windowed launch: blockIdx.y = source, largest facet first as in k_fit, one
// thread per position.  Blocks past a source's positions, and those of
// sources that k_window_knots takes, leave at once: the grid is sized for the
// largest possible box.
template <int R, bool kExact, bool kMixed>
__global__ __launch_bounds__(256) void k_fit_window(FitArgs a, int num_r) {
  const int s = a.size_order ? a.size_order[a.n_src - 1 - (int)blockIdx.y] : (int)blockIdx.y;
  const Window w(a, s);
  if (w.positions() <= a.knot_positions) return;
  const int j = w.point(a, blockIdx.x * blockDim.x + threadIdx.x);
  if (j >= 0) eval_point<R, kExact, kMixed>(a, num_r, s, j);
}

// The same for the sources of at most a.knot_positions positions, 64 per
// block, the knots shared by the block's four waves.  A narrowed fit is a few
// waves per source and the walk over the largest facet's records (some 900
// VALU cycles per record with all 20 knots in a lane) outlasts all others;
// shared knots make it four times shorter.  300 sources, us, k_fit_window |
// k_window_knots: lattice of every fourth point and its boxes 709 | 409, boxes
// of 9 x 9 points 269 | 122; 1000 sources 1,180 | 1,111 and 363 | 195.
template <bool kMixed>
__global__ __launch_bounds__((KnotSplit<kMixed, 0>::kThreads), (KnotSplit<kMixed, 0>::kWavesPerSimd)) void k_window_knots(
    FitArgs a, int num_r) {
  __shared__ double sh[block_doubles<0, KnotSplit<kMixed, 0>::kWaves>()];
  const int s = a.size_order ? a.size_order[a.n_src - 1 - (int)blockIdx.y] : (int)blockIdx.y;
  const Window w(a, s);
  if (w.positions() > a.knot_positions) return;
  const int j = w.point(a, blockIdx.x * 64 + (int)(threadIdx.x & 63));
  if (!__any(j >= 0)) return;                  // the same in every wave
  double L = NAN;
  if (a.offsets[s + 1] != a.offsets[s]) {      // uniform
    // a lane without a point evaluates the centre and drops it
    const int f = j >= 0 ? a.epts[j] : w.ctr * a.n_e + w.ctr;
    const int i1 = f / a.n_e, i2 = f - i1 * a.n_e;
    L = loglike_block<kMixed, 0, KnotSplit<kMixed, 0>::kWaves>(a, num_r, s, (double)(i1 - w.ctr) * a.e_step, (double)(i2 - w.ctr) * a.e_step, sh);
  }
  if (threadIdx.x < 64 && j >= 0) a.lsurf[(int64_t)s * a.n_valid + j] = L;
}

// Persistent work queue: a grid sized to the resident capacity; each wave
// claims items with one atomic; item -> (rank, piece) by binary search of the
// per-rank item offsets; a rank is a source (ranks ordered by decreasing cell
// count, so the longest items go first), a piece is tile*64 consecutive valid
// grid points.  Every wave leaves when the counter passes the item count.
template <int R, bool kExact, bool kMixed>
__global__ __launch_bounds__(256) void k_fit_queue(FitArgs a, QueueArgs q, int num_r) {
  const int lane = threadIdx.x & 63;
  for (;;) {
    uint32_t item = 0;
    if (lane == 0) item = atomicAdd(q.counter, 1u);
    item = __shfl(item, 0);
    if ((int64_t)item >= q.n_items) break;
    int lo = 0, hi = q.n_rank;                          // item_start[lo] <= item < item_start[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (q.item_start[mid] <= (int64_t)item) lo = mid;
      else hi = mid;
    }
    const int s = q.order[lo];
    const int tile = q.tile[lo];
    const int64_t piece = (int64_t)item - q.item_start[lo];
    for (int t = 0; t < tile; ++t) {
      const int64_t j = (piece * tile + t) * 64 + lane;
      if (j < a.n_valid) eval_point<R, kExact, kMixed>(a, num_r, s, (int)j);
    }
  }
}

// Window seeded by the stride-S lattice (after lattice pass 1): per source,
// the bounding box of the lattice points within the threshold of the lattice
// maximum, widened by S grid steps and clamped to the grid; the whole grid
// for an empty facet.  One wave per source.
__global__ __launch_bounds__(256) void k_lattice_windows(FitArgs a, double log_frac, int32_t *win) {
  const int lane = threadIdx.x & 63;
  const int s = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (s >= a.n_src) return;                                      // uniform per wave
  int4 *w = reinterpret_cast<int4 *>(win) + s;
  const int S = a.check_stride, ctr = (a.n_e - 1) / 2, h = ctr / S, nl = 2 * h + 1;
  const double *L = a.lsurf + (int64_t)s * a.n_valid;
  double best = -INFINITY;
  if (a.offsets[s + 1] > a.offsets[s]) {
    for (int u = lane; u < nl * nl; u += 64) {
      const int j = a.valid_index[(ctr + S * (u / nl - h)) * a.n_e + ctr + S * (u % nl - h)];
      if (j >= 0) best = fmax(best, L[j]);
    }
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) best = fmax(best, __shfl_xor(best, d));
  if (!(best > -INFINITY)) {
    if (lane == 0) *w = make_int4(0, a.n_e - 1, 0, a.n_e - 1);
    return;
  }
  const double thr = best + log_frac;
  int lo1 = a.n_e, hi1 = -1, lo2 = a.n_e, hi2 = -1;
  for (int u = lane; u < nl * nl; u += 64) {
    const int i1 = ctr + S * (u / nl - h), i2 = ctr + S * (u % nl - h);
    const int j = a.valid_index[i1 * a.n_e + i2];
    if (j >= 0 && L[j] >= thr) {
      lo1 = min(lo1, i1);
      hi1 = max(hi1, i1);
      lo2 = min(lo2, i2);
      hi2 = max(hi2, i2);
    }
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    lo1 = min(lo1, __shfl_xor(lo1, d));
    hi1 = max(hi1, __shfl_xor(hi1, d));
    lo2 = min(lo2, __shfl_xor(lo2, d));
    hi2 = max(hi2, __shfl_xor(hi2, d));
  }
  if (lane == 0)
    *w = make_int4(max(lo1 - S, 0), min(hi1 + S, a.n_e - 1), max(lo2 - S, 0), min(hi2 + S, a.n_e - 1));
}

__global__ void k_reset_counter(uint32_t *c) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *c = 0u;
}

#define RLF_FIT_DISPATCH(KERNEL, GRID, ...)                                                         \
  do {                                                                                              \
    if (a.num_r == 20)                                                                              \
      hipLaunchKernelGGL((KERNEL<20, true, kMixed>), GRID, dim3(256), 0, st, __VA_ARGS__, 20);     \
    else if (a.num_r == 23)                                                                         \
      hipLaunchKernelGGL((KERNEL<23, true, kMixed>), GRID, dim3(256), 0, st, __VA_ARGS__, 23);     \
    else if (a.num_r <= 8)                                                                          \
      hipLaunchKernelGGL((KERNEL<8, false, kMixed>), GRID, dim3(256), 0, st, __VA_ARGS__, a.num_r); \
    else                                                                                            \
      hipLaunchKernelGGL((KERNEL<kMaxKnots, false, kMixed>), GRID, dim3(256), 0, st, __VA_ARGS__,  \
                         a.num_r);                                                                  \
  } while (0)

// Mixed form: launches of more than kPosGroups groups of 64 points (15 sources
// on the 81 x 81 grid) take k_fit_pos.  16 sources, k_fit_knots | k_fit_pos: 3
// x 3 offsets 284 | 337 us, 5 x 5 546 | 732, 7 x 7 1,321 | 1,730; 32 sources
// 494 | 414, 939 | 911, 2,362 | 2,003; with facets of very different sizes the
// lines cross at 15 sources (3 x 3, 16 sources: 302 | 275).
constexpr int64_t kPosGroups = 1500;

template <bool kMixed, int NP>
hipError_t launch_knots(const FitArgs &a, hipStream_t st) {
  constexpr int threads = KnotSplit<kMixed, NP>::kThreads;
  if constexpr (kMixed && NP != 0)
    if ((a.n_valid + 63) / 64 * (int64_t)a.n_src > kPosGroups) {
      hipLaunchKernelGGL(k_fit_pos<NP>, dim3((a.n_valid + 255) / 256, a.n_src), dim3(256), 0, st, a, a.num_r);
      return hipGetLastError();
    }
  hipLaunchKernelGGL((k_fit_knots<kMixed, NP>), dim3((a.n_valid + 63) / 64, a.n_src), dim3(threads), 0, st, a, a.num_r);
  return hipGetLastError();
}

// Narrowed fits: k_window_knots takes the sources of at most this many
// positions.  Where a launch fills the card k_fit_window is the better one
// (its lanes form the quadratic form once instead of four times).  k_fit_window
// | k_window_knots, us, FP64 and mixed: 100 sources of 31 x 31 points 373 | 204
// and 392 | 233, 300 469 | 425 and 497 | 420, 600 671 | 721 and 730 | 751; 300 of 17
// x 17 373 | 187 and 412 | 234; whole grids of 40 405 | 362 and 413 | 346, of 80
// 672 | 706 and 656 | 645, of 150 1,170 | 1,237 and 1,113 | 1,120.  The boxes are on
// the device, so a launch whose boxes could fill the card is split by their
// size, two kernels each leaving the other's sources at once, up to the
// number of sources where the idle blocks cost more than that gains (2,000 of 3 x
// 3 points 390 and 470, split about 510 in FP64).  The lattice and the boxes it
// leads to are small: one kernel (every fourth point, 1,000 sources 1,139 |
// 1,081 and 1,278 | 1,188, 2,000 2,489 | 2,568 and 2,619 | 2,594).
constexpr int kLatticeSources = 1000, kKnotWindows = 80, kSplitWindows = 1500, kKnotWork = 400000;

int knot_positions(const FitArgs &a, int positions) {
  if (a.n_src <= (a.lattice_pass ? kLatticeSources : kKnotWindows)) return positions;
  return !a.lattice_pass && a.n_src <= kSplitWindows ? std::min(positions, kKnotWork / a.n_src) : 0;
}

// Blocks per source for up to n positions, an odd number: blocks go to the
// eight XCDs in turn by linear index, and with a multiple of eight the first
// blocks of all sources, often the only ones with work, sit on one of them
// (200 sources of 3 x 3 points: 342 us with 32 blocks, 119 with 33; the lattice fit of 2,000 sources
// with 26 blocks 2,903, with 27 2,370).
unsigned odd_blocks(int n, int per) { return (unsigned)((n + per - 1) / per) | 1u; }

template <bool kMixed>
hipError_t launch(const FitArgs &a, hipStream_t st) {
  if (a.n_pos) {
    if (a.window || a.lattice_pass) return hipErrorInvalidValue;   // full grid only
    if (a.n_pos == 9) return launch_knots<kMixed, 9>(a, st);
    if (a.n_pos == 25) return launch_knots<kMixed, 25>(a, st);
    if (a.n_pos == 49) return launch_knots<kMixed, 49>(a, st);
    return hipErrorInvalidValue;
  }
  if (a.window || a.lattice_pass == 1) {
    const int h = a.check_stride > 0 ? ((a.n_e - 1) / 2) / a.check_stride : 0;
    const int lattice = (a.check_stride > 0 && a.lattice_pass != 2) ? (2 * h + 1) * (2 * h + 1) : 0;
    const int positions = (a.lattice_pass == 1 ? 0 : a.n_e * a.n_e) + lattice;
    FitArgs w = a;
    w.knot_positions = knot_positions(a, positions);
    if (w.knot_positions < positions) RLF_FIT_DISPATCH(k_fit_window, dim3(odd_blocks(positions, 256), a.n_src), w);
    if (w.knot_positions > 0)
      hipLaunchKernelGGL(k_window_knots<kMixed>, dim3(odd_blocks(std::min(positions, w.knot_positions), 64), a.n_src),
                         dim3(KnotSplit<kMixed, 0>::kThreads), 0, st, w, a.num_r);
  } else if (a.redo || (a.n_valid + 63) / 64 * (int64_t)a.n_src <= kKnotGroups) {
    return launch_knots<kMixed, 0>(a, st);
  } else {
    RLF_FIT_DISPATCH(k_fit, dim3((a.n_valid + 255) / 256, a.n_src), a);
  }
  return hipGetLastError();
}

template <bool kMixed>
hipError_t launch_q(const FitArgs &a, const QueueArgs &q, int blocks, hipStream_t st) {
  hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(64), 0, st, q.counter);
  RLF_FIT_DISPATCH(k_fit_queue, dim3(blocks), a, q);
  return hipGetLastError();
}

template <bool kMixed>
int queue_blocks_per_cu(int num_r) {
  int n = 0;
  hipError_t e;
  if (num_r == 20) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_fit_queue<20, true, kMixed>, 256, 0);
  else if (num_r == 23) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_fit_queue<23, true, kMixed>, 256, 0);
  else if (num_r <= 8) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_fit_queue<8, false, kMixed>, 256, 0);
  else e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_fit_queue<kMaxKnots, false, kMixed>, 256, 0);
  return (e == hipSuccess && n > 0) ? n : 1;
}

}  // namespace

hipError_t launch_fit_f64(const FitArgs &a, hipStream_t st) { return launch<false>(a, st); }
hipError_t launch_fit_mixed(const FitArgs &a, hipStream_t st) { return launch<true>(a, st); }

namespace {

template <bool kMixed, int NP>
hipError_t refine_eval(const FitArgs &a, const RefineArgs &r, hipStream_t st) {
  hipLaunchKernelGGL((k_refine_eval<kMixed, NP>), dim3(odd_blocks(r.max_side * r.max_side, 64), a.n_src), dim3(64 * refine_waves<kMixed, NP>()), 0,
                     st, a, r, a.num_r);
  return hipGetLastError();
}

template <bool kMixed>
hipError_t refine_eval(const FitArgs &a, const RefineArgs &r, hipStream_t st) {
  switch (a.n_pos) {
    case 0: return refine_eval<kMixed, 0>(a, r, st);
    case 9: return refine_eval<kMixed, 9>(a, r, st);
    case 25: return refine_eval<kMixed, 25>(a, r, st);
    case 49: return refine_eval<kMixed, 49>(a, r, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_refine_eval(const FitArgs &a, const RefineArgs &r, int mixed, hipStream_t st) {
  return mixed ? refine_eval<true>(a, r, st) : refine_eval<false>(a, r, st);
}

hipError_t launch_lattice_windows(const FitArgs &a, double log_frac, int32_t *win, hipStream_t st) {
  if (a.check_stride < 2) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_lattice_windows, dim3((a.n_src + 3) / 4), dim3(256), 0, st, a, log_frac, win);
  return hipGetLastError();
}

hipError_t launch_fit_queue(const FitArgs &a, const QueueArgs &q, int mixed, int blocks, hipStream_t st) {
  if (a.n_pos) return hipErrorInvalidValue;                      // position fixed only
  return mixed ? launch_q<true>(a, q, blocks, st) : launch_q<false>(a, q, blocks, st);
}

int fit_queue_blocks_per_cu(int mixed, int num_r) {
  return mixed ? queue_blocks_per_cu<true>(num_r) : queue_blocks_per_cu<false>(num_r);
}

}  // namespace rlf
