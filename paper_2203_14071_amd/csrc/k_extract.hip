// Facet extraction (Sec. 2.3): per (visibility, source) pair, phase-shift the
// residual to the source, add back the source's own model, and accumulate the
// weighted result into the source's facet cell (rint(u theta), rint(v theta)).
//
// Work decomposition.  Lanes are sources: a wave holds 64 NS sources (NS per
// lane, their constants in VGPRs; lane slots take the sources in order of
// facet cell size, so the cell changes of a wave's lanes tend to coincide
// and the branches diverge less) and walks a chunk of visibilities in the
// facet object's uv-sorted order; each visibility's data is uniform across
// the wave and arrives through scalar loads.  Along the sorted order a
// source stays in one facet cell for runs of ~100-300 visibilities and,
// near a cell boundary, alternates between the same two cells many times
// (a Morton curve crosses a boundary back and forth).  Each lane therefore
// keeps two runs (count, W, Z) in registers, its current cell's and the
// previous cell's, swaps them when it returns to the previous cell, and
// issues global atomics only when it enters a third cell or the chunk ends:
// on the 1000-source SKA-MID field one atomic flush per ~20 cell changes
// (with one run per lane, every cell change flushed), and no cross-lane
// merging is needed.
//
// XCD-aware launch: blocks are dispatched round-robin over the 8 XCDs; the
// grid is laid out so that all blocks of one visibility chunk (all source
// tiles) land on one XCD and share its L2 for the chunk's data.
//
// Integer results are exact (cell index in FP64 exactly as rint(fl(u theta)));
// FP sums are atomic and order-dependent in their last bits.  Runs are summed
// in FP64 in both forms (the mixed form's FP32 terms are widened per term).
#include <algorithm>

#include "rlf_devmath.h"
#include "rlf_internal.h"
#include "rlf_lanes.h"
#include "rlf_launch.h"
#include "rlf_sky.h"

namespace rlf {

namespace {

constexpr int kXcd = 8;
// Waves per block of k_extract by the entries T of the FP64 form's table (the
// mixed form has none): 2048 take 32 KB of LDS, so that four blocks of 8 waves per
// CU keep eight waves per SIMD; 1024 take 16 KB, eight blocks of 4 (run_tiles).
template <bool kMixed, int T>
constexpr int waves_per_block() { return kMixed || T == 1024 ? 4 : 8; }
constexpr int kNsF64 = 1, kNsMixed = 1;        // sources per lane
constexpr int kGroupF64 = 2, kGroupMixed = 4;  // visibilities whose scalar loads are issued together
constexpr double kNoRun = 1099511627776.0;    // 2^40: "no open run" (run keys are below 2^31 in magnitude)
constexpr int32_t kNoKey = INT32_MIN;          // the same for the previous run's integer key

// Catalogues of at most kVpSources sources go through k_extract_vp, larger
// ones through k_extract: its lanes are sources, and with few tiles a chunk's
// scalar loads are shared by few waves.  k_extract | k_extract_vp, us: 1,158,361
// visibilities, 130, 160 and 192 sources FP64 443 | 394, 475 | 448 and 510 | 510,
// 160, 192 and 256 mixed 405 | 354, 407 | 397 and 467 | 480; 5,000,000, 160, 192
// and 256 FP64 1,717 | 1,513, 1,771 | 1,769 and 2,137 | 2,317, 192 and 256 mixed
// 1,227 | 1,195 and 1,505 | 1,556.
constexpr int kVpSourcesF64 = 160, kVpSourcesMixed = 192;
// ... and so do launches that would leave the chip idle through k_extract:
// fewer than kTileWaves waves of kMinChunk visibilities (11,400 visibilities,
// 100 sources: 156 us against 37; 240,000 and 640, 9,380 waves, FP64 402 | 354,
// mixed 297 | 282; 800,000 and 256, 12,500, 486 | 453 and 357 | 347; 500,000 and
// 448, 13,678, FP64 460 | 513).  Its waves take two sources at a time, each
// at least a step of 64 visibilities, two reductions and eight atomics, so
// large catalogues go the other way.  k_extract | k_extract_vp, us: 11,400
// visibilities, 1,000, 1,200 and 4,000 sources FP64 179 | 137, 173 | 178 and
// 351 | 692, mixed 106 | 113, 123 | 130 and 314 | 622; 20,000, 800 and 2,000
// FP64 122 | 84 and 184 | 216, mixed 92 | 76 and 149 | 180; 2,000, 2,000 and
// 10,000 FP64 178 | 92 and 250 | 991, mixed 89 | 80 and 239 | 893.
constexpr int64_t kMinChunk = 256, kTileWaves = 12600;
constexpr int64_t kVpCatalogueF64 = 1024, kVpCatalogueMixed = 800;
// ... the larger of them only where there are enough visibilities for the steps
// and few enough waves for the tiles (30,000 and 1,500 FP64 185 | 168, mixed 159 |
// 148; 20,000 and 1,500 145 | 158 and 114 | 120; 150,000 and 1,000 mixed 351 | 309,
// 200,000 and 1,000, 12,512 waves, 390 | 430), or where all is small (600 and 3,000
// FP64 116 | 85, mixed 86 | 73; 2,000 and 3,000 mixed 96 | 135).
constexpr int64_t kVpCatalogueLarge = 1536, kVpLargeVis = 25000, kVpLargeWaves = 10400;
constexpr int64_t kVpCatalogueTiny = 3072, kTinyPairs = 4000000;

bool visibilities_on_lanes(int64_t n_vis, int64_t n_src, int mixed) {
  if (n_src <= (mixed ? kVpSourcesMixed : kVpSourcesF64)) return true;
  const int64_t waves = (n_vis + kMinChunk - 1) / kMinChunk * ((n_src + 63) / 64);
  if (waves >= kTileWaves) return false;
  if (n_src <= (mixed ? kVpCatalogueMixed : kVpCatalogueF64)) return true;
  if (n_src <= kVpCatalogueLarge && n_vis >= kVpLargeVis && waves < kVpLargeWaves) return true;
  return n_src <= kVpCatalogueTiny && n_vis * n_src <= kTinyPairs;
}

// Work item of a wave: blocks go to the eight XCDs round-robin by index; item
// (chunk, part) with the parts of a chunk (source tiles or groups, which read
// the same visibilities) side by side on one XCD, and consecutive chunks on
// consecutive XCDs, so that every XCD gets its share of the dense and of the
// sparse regions of the plane (a contiguous eighth of the order per XCD
// measured 3 % slower on the 1000-source field).
struct WorkItem {
  int64_t chunk;
  int part;
};
__device__ __forceinline__ WorkItem work_item(int waves, int parts) {
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t w = (blockIdx.x / kXcd) * waves + wid;           // wave within its XCD
  const uint32_t c = w / (uint32_t)parts;
  return WorkItem{(int64_t)c * kXcd + blockIdx.x % kXcd, (int)(w - c * (uint32_t)parts)};
}

// One source of a lane: facet geometry and two open runs, the current cell's
// and the cell the lane was in before it.  Near a cell boundary the sorted
// order crosses back and forth between the same two cells many times, so a
// return to the previous cell only swaps the two runs; global memory is
// touched when a third cell is entered (the older run is flushed) and at
// the end of the chunk.  A run key is iy * side + ix (an exact integer in
// FP64); base already holds the offset half * (side + 1) of cell (0, 0) in
// the source's dense block.  Counts are kept relative to the
// lane-independent count nproc of processed visibilities: the current run
// holds nproc - cb visibilities, the other run ocnt.
struct LaneSrc {
  bool active;
  int32_t half;
  int64_t base;
  double side;
  double key, rw, rzr, rzi;        // current cell
  double ow, ozr, ozi;             // the cell before it
  int32_t okey, cb, ocnt;          // okey: the previous cell's key, or kNoKey
};

// Add a run to its dense cell: four FP64 atomics at one address (the count
// is an exact integer in FP64).
__device__ __forceinline__ void flush(double4 *__restrict__ acc, int64_t base, int32_t key, double w, double zr,
                                      double zi, int32_t n) {
  double *c = &acc[base + key].x;
  unsafeAtomicAdd(c, w);
  unsafeAtomicAdd(c + 1, zr);
  unsafeAtomicAdd(c + 2, zi);
  unsafeAtomicAdd(c + 3, (double)n);
}

// Run bookkeeping of one lane source at one visibility (nproc = visibilities
// of the chunk with weight > 0 processed before this one, uniform).  When
// the cell changes: back to the previous cell swaps the two runs; a new cell
// flushes the older run, demotes the current one and opens an empty run
// (after the bounds check).  The caller then adds the visibility's terms to
// the current run.
__device__ __forceinline__ void enter_cell(LaneSrc &L, double4 *__restrict__ acc, uint32_t *err, int32_t nproc,
                                           double xf, double yf) {
  const double k = fma(yf, L.side, xf);
  if (k != L.key) {
    const int32_t tk = L.key == kNoRun ? kNoKey : (int32_t)L.key;
    const double tw = L.rw, tr = L.rzr, ti = L.rzi;
    const int32_t tn = nproc - L.cb;
    if (L.okey != kNoKey && k == (double)L.okey) {
      L.key = (double)L.okey;
      L.rw = L.ow;
      L.rzr = L.ozr;
      L.rzi = L.ozi;
      L.cb = nproc - L.ocnt;
    } else {
      if (L.okey != kNoKey && L.active) flush(acc, L.base, L.okey, L.ow, L.ozr, L.ozi, L.ocnt);
      const double half = (double)L.half;
      const bool inb = fabs(xf) <= half && fabs(yf) <= half;
      if (!inb && L.active) atomicOr(err, 1u);
      L.key = inb ? k : kNoRun;
      L.cb = nproc;
      L.rw = L.rzr = L.rzi = 0.0;
    }
    L.okey = tk;
    L.ow = tw;
    L.ozr = tr;
    L.ozi = ti;
    L.ocnt = tn;
  }
}

// The read-only visibility data and the atomic targets are separate
// restrict-qualified kernel parameters: with no possible aliasing the
// compiler keeps the per-visibility loads scalar (s_load) although the loop
// issues atomics.  Per visibility the wave loads (u, v, w, spec), the
// profile's quadratic terms, the residual and the weight (FP64 form: the
// weighted residual w R and w spec, so that the run sums take the shifted
// residual and the own model in three FMAs and two); flagged visibilities
// carry weight +0 and are skipped on a scalar test of the bits.
// A lane may hold NS sources (NS * 64 per wave) to share each load.
//
// Cell index: ix = rint(fl(u theta)) and iy likewise, in FP64 (exact
// integers); the run key iy side + ix is formed in FP64 too (one FMA, exact:
// |key| < 2^31) and compared as a double, so the common path has no
// conversions.  The facet half-size was sized on the host from the largest
// |u|, |v| with the same rounding chain, so every index is inside its facet;
// the bound is still checked whenever a new cell's run starts (err bit 0).
//
// Occupancy: the FP64 form is held to 64 VGPRs (eight waves per SIMD; the
// few values that spill, the lane's dense-block base among them, are
// reloaded only on the rare third-cell flush and after the loop), the mixed
// form fits eight waves by itself (51 VGPRs) under any bound; its bound
// steers the scalar registers: a minimum of 7 waves gives 94 SGPRs with two
// spilled to VGPR lanes and measured 4.5 % faster than 6 (97 SGPRs, none
// spilled), while 8 spills 17 and is 15 % slower.
template <bool kMixed, int NS, int G, int T>
__global__ __launch_bounds__((64 * waves_per_block<kMixed, T>()), kMixed ? 7 : 8) void k_extract(
    ExtractArgs a, const double4 *__restrict__ sgeo, const void *__restrict__ squad, const void *__restrict__ sres,
    const uint64_t *__restrict__ swt, double4 *__restrict__ acc) {
  constexpr int kW = waves_per_block<kMixed, T>();
  __shared__ double2 tab[kMixed ? 1 : T];
  if (!kMixed) {
    cis_table_load<T>(tab, a.cis);
    __syncthreads();
  }
  const int lane = threadIdx.x & 63;
  const WorkItem it = work_item(kW, a.n_tiles);
  const int64_t chunk = it.chunk;
  const int tile = it.part;
  if (chunk >= a.n_chunks) return;                               // uniform per wave

  LaneSrc L[NS];
  int src[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int s_raw = (tile * NS + i) * 64 + lane;
    L[i].active = s_raw < a.n_src;
    src[i] = a.order[L[i].active ? s_raw : a.n_src - 1];
    const SrcGeom g = a.geom[src[i]];
    L[i].base = g.base + (int64_t)g.half * (g.side + 1);
    L[i].half = g.half;
    L[i].side = (double)g.side;
    L[i].key = kNoRun;
    L[i].okey = kNoKey;
    L[i].cb = L[i].ocnt = 0;
    L[i].rw = L[i].rzr = L[i].rzi = 0.0;
    L[i].ow = L[i].ozr = L[i].ozi = 0.0;
  }
  int32_t nproc = 0;
  const int64_t j0 = chunk * (int64_t)a.chunk;
  const int len = (int)(min(a.sv.n_vis, j0 + (int64_t)a.chunk) - j0);
  const double4 *__restrict__ geo = sgeo + j0;
  const uint64_t *__restrict__ wt = swt + j0;                    // weight bits: 0 = skip

  if (!kMixed) {
    // the flux folded into the profile argument: with x' = c0 x and
    // c0 = (3/2 S)^{-2/3}, pow_m32_f64(x') = (2/3) x'^{-3/2} = S x^{-3/2},
    // the own model per unit spectral factor, with no multiplication by S
    // per pair (S = 0: c0 = 1e250, x' >= 1e250 and the term underflows to
    // exactly zero; c0 finite, so no infinity meets a zero coefficient)
    SrcModel p[NS];
    double c0[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      p[i] = a.src[src[i]];
      c0[i] = p[i].flux > 0.0 ? pow(kPowM32Scale * p[i].flux, -2.0 / 3.0) : 1e250;
      p[i].q11 *= c0[i];
      p[i].q12x2 *= c0[i];
      p[i].q22 *= c0[i];
    }
    const double4 *__restrict__ quad = reinterpret_cast<const double4 *>(squad) + j0;
    const double2 *__restrict__ res = reinterpret_cast<const double2 *>(sres) + j0;
    for (int jl = 0; jl < len; jl += G) {
      double4 gg[G], qg[G];
      double2 rg[G];
      uint64_t wwg[G];
#pragma unroll
      for (int t = 0; t < G; ++t) {
        gg[t] = geo[jl + t];
        qg[t] = quad[jl + t];
        rg[t] = res[jl + t];
        wwg[t] = wt[jl + t];
      }
      // the group's values are needed here: the loads the compiler would
      // otherwise sink past the weight test below (a second round trip to
      // memory per group) are issued together with the others
#pragma unroll
      for (int t = 0; t < G; ++t)
        asm volatile("" ::"s"(gg[t].x), "s"(gg[t].y), "s"(gg[t].z), "s"(qg[t].x), "s"(qg[t].y), "s"(qg[t].z));
#pragma unroll
      for (int t = 0; t < G; ++t) {
        if (jl + t >= len) break;                                   // uniform
        if (wwg[t] == 0u) continue;                                  // uniform: flagged or padding
        const double u = gg[t].x, v = gg[t].y, ww = __longlong_as_double((long long)wwg[t]);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
          const double ph = fma(u, p[i].l, fma(v, p[i].m, gg[t].z * p[i].n1));
          const double2 cs = cis2pi_f64<T>(ph, tab);
          const double x = fma(p[i].q11, qg[t].x, fma(p[i].q12x2, qg[t].y, fma(p[i].q22, qg[t].z, c0[i])));
          const double own = pow_m32_f64(x);                        // own model / spec, real after the shift
          enter_cell(L[i], acc, a.err, nproc, rint(__dmul_rn(u, p[i].theta)), rint(__dmul_rn(v, p[i].theta)));
          // w z = (w R) exp(-2 pi i ph) + (w spec) own
          L[i].rw += ww;
          L[i].rzr = fma(rg[t].x, cs.x, fma(rg[t].y, cs.y, fma(qg[t].w, own, L[i].rzr)));
          L[i].rzi = fma(rg[t].y, cs.x, fma(-rg[t].x, cs.y, L[i].rzi));
        }
        ++nproc;
      }
    }
  } else {
    // (the flux stays a multiplication here: folded into the profile
    // argument as in the FP64 form it saves an instruction per pair but
    // measured 0.6 % slower on the 10,000-source field, and again 0.8 %
    // slower on the 1000-source field with the kernel as it is now)
    SrcMixed p[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) p[i] = a.src32[src[i]];
    const float4 *__restrict__ quad = reinterpret_cast<const float4 *>(squad) + j0;
    const float2 *__restrict__ res = reinterpret_cast<const float2 *>(sres) + j0;
    for (int jl = 0; jl < len; jl += G) {
      double4 gg[G];
      float4 qg[G];
      float2 rg[G];
      uint64_t wwg[G];
#pragma unroll
      for (int t = 0; t < G; ++t) {
        gg[t] = geo[jl + t];
        qg[t] = quad[jl + t];
        rg[t] = res[jl + t];
        wwg[t] = wt[jl + t];
      }
      // the group's values are needed here: the loads the compiler would
      // otherwise sink past the weight test below (a second round trip to
      // memory per group) are issued together with the others
#pragma unroll
      for (int t = 0; t < G; ++t)
        asm volatile("" ::"s"(gg[t].x), "s"(gg[t].y), "s"(gg[t].z), "s"(qg[t].x), "s"(qg[t].y), "s"(qg[t].z));
#pragma unroll
      for (int t = 0; t < G; ++t) {
        if (jl + t >= len) break;                                   // uniform
        if (wwg[t] == 0u) continue;                                  // uniform: flagged or padding
        const double u = gg[t].x, v = gg[t].y, ww = __longlong_as_double((long long)wwg[t]);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
          const double ph = fma(u, p[i].l, fma(v, p[i].m, gg[t].z * p[i].n1));
          const float tt = (float)__builtin_amdgcn_fract(ph);        // turns, in [0, 1]
          const float sn = __builtin_amdgcn_sinf(tt), cs = __builtin_amdgcn_cosf(tt);
          float zr = fmaf(rg[t].x, cs, rg[t].y * sn);
          const float zi = fmaf(rg[t].y, cs, -(rg[t].x * sn));
          const float x = fmaf(p[i].q11, qg[t].x, fmaf(p[i].q12x2, qg[t].y, fmaf(p[i].q22, qg[t].z, 1.0f)));
          const float q = __builtin_amdgcn_rsqf(x);
          zr = fmaf(qg[t].w * p[i].flux, q * q * q, zr);
          enter_cell(L[i], acc, a.err, nproc, rint(__dmul_rn(u, p[i].theta)), rint(__dmul_rn(v, p[i].theta)));
          L[i].rw += ww;
          L[i].rzr = fma(ww, (double)zr, L[i].rzr);
          L[i].rzi = fma(ww, (double)zi, L[i].rzi);
        }
        ++nproc;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    if (!L[i].active) continue;
    if (L[i].key != kNoRun) flush(acc, L[i].base, (int32_t)L[i].key, L[i].rw, L[i].rzr, L[i].rzi, nproc - L[i].cb);
    if (L[i].okey != kNoKey) flush(acc, L[i].base, L[i].okey, L[i].ow, L[i].ozr, L[i].ozi, L[i].ocnt);
  }
}

// Visibility-parallel extraction: small catalogues, small observations, the
// chunks of a sequential refinement (visibilities_on_lanes).  A wave takes
// a.chunk steps of 64 consecutive sorted visibilities, one per lane (coalesced
// loads, the next step's issued before this one's arithmetic), for NS sources at a time
// (their records wave-uniform, so the loads serve both), and evaluates each
// pair exactly as k_extract does.  Along the sorted order a source stays in
// one facet cell for runs of ~200 visibilities and alternates between two
// cells near a boundary, so the wave keeps two open cells per source whose
// keys are wave-uniform and whose sums are per-lane partial sums: a step that
// falls into one open cell (about three in four) costs three additions, a
// step split between them a masked set of each, and only a third cell makes
// the wave reduce the less recent one over its lanes and add it to memory
// (four FP64 atomics).  A segmented scan over the lanes at every step would cost
// about four times the pair arithmetic.
__device__ __forceinline__ double from_lane(double x, int l) {   // l wave-uniform
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                          __builtin_amdgcn_readlane(__double2loint(x), l));
}

// x + x of the lane kRor below in the row of 16 (cyclic), by DPP (a VALU
// operand modifier: no LDS round trip).
template <int kRor>
__device__ __forceinline__ double add_ror(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x120 + kRor, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x120 + kRor, 0xf, 0xf, false);
  return x + __hiloint2double(hi, lo);
}

// An open cell of a wave: wave-uniform run key (kNoRun: none) and count, the
// lanes' partial sums.
struct OpenCell {
  double key;
  int32_t n;
  double w, zr, zi;
  __device__ __forceinline__ void open(double k) {
    key = k;
    n = 0;
    w = zr = zi = 0.0;
  }
  // Add on the lanes of m, all 64 lanes active: three additions under an
  // execution mask (written as selects, the compiler spends six more
  // instructions and copies of all sums where the branches join).
  __device__ __forceinline__ void add(uint64_t m, double vw, double vr, double vi) {
    asm volatile("s_mov_b64 exec, %6\n\tv_add_f64 %0, %0, %3\n\tv_add_f64 %1, %1, %4\n\tv_add_f64 %2, %2, %5\n\t"
                 "s_mov_b64 exec, -1"
                 : "+v"(w), "+v"(zr), "+v"(zi)
                 : "v"(vw), "v"(vr), "v"(vi), "s"(m));
    n += __popcll(m);
  }
  // Reduce over the lanes and add to the dense cell: row r of 16 lanes ends
  // up with component r, and its first lane issues one FP64 atomic (four
  // consecutive addresses).
  __device__ __forceinline__ void close(double4 *__restrict__ acc, int64_t base, int lane) const {
    if (key == kNoRun) return;                                   // uniform
    const double cnt = lane == 0 ? (double)n : 0.0;
    double x = fold_lanes<false>(fold_lanes<true>(w, zi), fold_lanes<true>(zr, cnt));
    // rows 0, 1: w, zr; rows 2, 3: zi, count
    x = add_ror<8>(x);
    x = add_ror<4>(x);
    x = add_ror<2>(x);
    x = add_ror<1>(x);
    if ((lane & 15) == 0) unsafeAtomicAdd(&acc[base + (int32_t)key].x + (lane >> 4), x);
  }
};

__device__ __forceinline__ double uniform(double x) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(x)),
                          __builtin_amdgcn_readfirstlane(__double2loint(x)));
}

constexpr int kVpTable = 1024;
constexpr int kVpThreads = 256;

// kUpd (NS = 1, one source in the launch): the residual kept in sorted order
// is first updated for changed source models (UpdateArgs, as k_update_sorted
// does, with the same sums), in the same pass: each lane updates its
// visibilities and extracts from the updated values.
template <bool kMixed, int NS, bool kUpd>
__global__ __launch_bounds__(kVpThreads) void k_extract_vp(ExtractArgs a, const double4 *__restrict__ sgeo,
                                                           const void *sres, const uint64_t *__restrict__ swt,
                                                           double4 *__restrict__ acc, UpdateArgs u) {
  static_assert(!kUpd || NS == 1, "the update is fused for one source");
  __shared__ double2 tab[kMixed ? 1 : kVpTable];
  if (!kMixed) {
    cis_table_load<kVpTable>(tab, a.cis);
    __syncthreads();
  }
  const int lane = threadIdx.x & 63;
  const int groups = (a.n_src + NS - 1) / NS;
  const WorkItem it = work_item(kVpThreads / 64, groups);
  const int64_t jw = it.chunk * a.chunk * 64;
  if (jw >= a.sv.n_vis) return;                                  // uniform per wave
  const int first = it.part * NS;
  const int steps = (int)min((int64_t)a.chunk, (a.sv.n_vis - jw + 63) >> 6);

  SrcModel p[NS];
  SrcMixed pm[NS];
  int64_t base[NS];
  double half[NS], side[NS];
  OpenCell A[NS], B[NS];
  bool last_b[NS];                                               // uniform: the last visibility went to B
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    // a group past the last source repeats it without adding anything
    const int s = __builtin_amdgcn_readfirstlane(a.order[min(first + i, a.n_src - 1)]);
    if (kMixed) pm[i] = a.src32[s];
    else p[i] = a.src[s];
    const SrcGeom gm = a.geom[s];
    base[i] = gm.base + (int64_t)gm.half * (gm.side + 1);
    half[i] = (double)gm.half;
    side[i] = (double)gm.side;
    A[i].open(kNoRun);
    B[i].open(kNoRun);
    last_b[i] = false;
  }
  const bool two = NS == 1 || first + 1 < a.n_src;               // uniform
  double own_scale[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) own_scale[i] = kMixed ? 0.0 : uniform(kPowM32Scale * p[i].flux);

  // one visibility's data; element o of the wave's span (32-bit byte offsets
  // from wave-uniform pointers)
  struct Vis {
    double4 g;
    uint64_t w;
    double2 rd;
    float2 rf;
  };
  const char *gp = reinterpret_cast<const char *>(sgeo + jw), *wp = reinterpret_cast<const char *>(swt + jw);
  const char *rp = reinterpret_cast<const char *>(sres) + jw * (kMixed ? sizeof(float2) : sizeof(double2));
  auto load = [&](uint32_t o) {
    Vis x{};
    x.g = *reinterpret_cast<const double4 *>(gp + o * 32u);
    x.w = *reinterpret_cast<const uint64_t *>(wp + o * 8u);
    if (kMixed) x.rf = *reinterpret_cast<const float2 *>(rp + o * 8u);
    else if (!kUpd) x.rd = *reinterpret_cast<const double2 *>(rp + o * 16u);
    return x;
  };
  auto step = [&](const Vis &cur, uint32_t o) {
    const double4 gg = cur.g;
    const uint64_t wb = cur.w;
    double2 rd = cur.rd;
    float2 rf = cur.rf;

    const double ww = __longlong_as_double((long long)wb);
    double uu = 0.0, uv = 0.0, vv = 0.0, ws = 0.0;
    float uuf = 0.0f, uvf = 0.0f, vvf = 0.0f;
    const float spf = (float)gg.w;
    if (kMixed) {
      const float uf = (float)gg.x, vf = (float)gg.y;
      uuf = uf * uf;
      uvf = uf * vf;
      vvf = vf * vf;
    } else {
      uu = __dmul_rn(gg.x, gg.x);
      uv = __dmul_rn(gg.x, gg.y);
      vv = __dmul_rn(gg.y, gg.y);
      ws = __dmul_rn(ww, gg.w);
    }
    if (kUpd && jw + o < a.sv.n_vis) {
      const int64_t j = jw + o;
      if (!kMixed) {
        const double2 ao = sum_f64(gg.x, gg.y, gg.z, u.old64, 0, u.n_old, tab);
        const double2 an = sum_f64(gg.x, gg.y, gg.z, u.new64, 0, u.n_new, tab);
        double2 r = u.rs[j];
        r = make_double2(fma(gg.w, ao.x, r.x), fma(gg.w, ao.y, r.y));
        r = make_double2(fma(-gg.w, an.x, r.x), fma(-gg.w, an.y, r.y));
        u.rs[j] = r;
        rd = make_double2(ww * r.x, ww * r.y);
        reinterpret_cast<double2 *>(u.sv.res)[j] = rd;
      } else {
        const float2 ao = sum_mixed(gg.x, gg.y, gg.z, u.old32, 0, u.n_old);
        const float2 an = sum_mixed(gg.x, gg.y, gg.z, u.new32, 0, u.n_new);
        rf = make_float2(fmaf(spf, ao.x, rf.x), fmaf(spf, ao.y, rf.y));
        rf = make_float2(fmaf(-spf, an.x, rf.x), fmaf(-spf, an.y, rf.y));
        reinterpret_cast<float2 *>(u.sv.res)[j] = rf;
      }
    }
    const uint64_t all = __ballot(wb != 0u);                     // flagged and padding entries take no part
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      if (i > 0 && !two) break;                                  // uniform
      double zr, zi, xf, yf;
      if (!kMixed) {
        const double ph = fma(gg.x, p[i].l, fma(gg.y, p[i].m, gg.z * p[i].n1));
        const double2 cs = cis2pi_f64<kVpTable>(ph, tab);
        const double x = fma(p[i].q11, uu, fma(p[i].q12x2, uv, fma(p[i].q22, vv, 1.0)));
        const double own = own_scale[i] * pow_m32_f64(x);
        // w z = (w R) exp(-2 pi i ph) + (w spec) own
        zr = fma(rd.x, cs.x, fma(rd.y, cs.y, ws * own));
        zi = fma(rd.y, cs.x, -rd.x * cs.y);
        xf = rint(__dmul_rn(gg.x, p[i].theta));
        yf = rint(__dmul_rn(gg.y, p[i].theta));
      } else {
        const double ph = fma(gg.x, pm[i].l, fma(gg.y, pm[i].m, gg.z * pm[i].n1));
        const float tt = (float)__builtin_amdgcn_fract(ph);
        const float sn = __builtin_amdgcn_sinf(tt), cs = __builtin_amdgcn_cosf(tt);
        float fr = fmaf(rf.x, cs, rf.y * sn);
        const float fi = fmaf(rf.y, cs, -(rf.x * sn));
        const float x = fmaf(pm[i].q11, uuf, fmaf(pm[i].q12x2, uvf, fmaf(pm[i].q22, vvf, 1.0f)));
        const float qr = __builtin_amdgcn_rsqf(x);
        fr = fmaf(spf * pm[i].flux, qr * qr * qr, fr);
        zr = ww * (double)fr;
        zi = ww * (double)fi;
        xf = rint(__dmul_rn(gg.x, pm[i].theta));
        yf = rint(__dmul_rn(gg.y, pm[i].theta));
      }
      const double key = fma(yf, side[i], xf);
      uint64_t pend = all;
      for (;;) {                                                 // uniform; nearly always one round
        const uint64_t ma = __ballot(key == A[i].key) & pend, mb = __ballot(key == B[i].key) & pend;
        A[i].add(ma, ww, zr, zi);
        B[i].add(mb, ww, zr, zi);
        if (ma | mb) last_b[i] = (mb >> (63 - __clzll((long long)(ma | mb)))) & 1;
        pend &= ~(ma | mb);
        if (!pend) break;
        // the first lane left opens its cell in place of the less recent one
        const int l = __ffsll((unsigned long long)pend) - 1;
        if (!(fabs(from_lane(xf, l)) <= half[i] && fabs(from_lane(yf, l)) <= half[i])) {
          // out of the facet: a NaN coordinate (which equals no key, its own
          // included: it must not open a cell), or uvw changed
          if (lane == 0) atomicOr(a.err, 1u);
          pend &= ~(1ull << l);
          if (!pend) break;
          continue;
        }
        const double nk = from_lane(key, l);
        if (!last_b[i]) {
          const OpenCell x = A[i];
          A[i] = B[i];
          B[i] = x;
        }
        A[i].close(acc, base[i], lane);
        A[i].open(nk);
        last_b[i] = false;
      }
    }
  };
  // two steps per iteration, the loads of a step issued one step ahead (the
  // arrays are padded by two steps of zero weight, which take no part)
  uint32_t o = lane;
  Vis v0 = load(o);
  for (int t = 0; t < steps; t += 2, o += 128) {
    const Vis v1 = load(o + 64);
    step(v0, o);
    v0 = load(o + 128);
    if (t + 1 < steps) step(v1, o + 64);
  }
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    if (i > 0 && !two) break;
    A[i].close(acc, base[i], lane);
    B[i].close(acc, base[i], lane);
  }
}

// Chunks of a launch that has few of them: they go to the XCDs in turn, so that
// a number that is no multiple of eight leaves some XCDs a chunk more than the
// others.
constexpr int64_t kFewChunks = 64;
int64_t even_chunks(int64_t chunks) {
  return chunks > kXcd && chunks < kFewChunks ? (chunks + kXcd - 1) / kXcd * kXcd : chunks;
}

// Visibilities per wave of k_extract.  A wave's start and end cost its lanes two
// open runs each (eight atomics), so that few visibilities per wave are slow,
// and a chunk of the dense core of the plane takes longer than one of its
// outskirts, which only many waves even out: 1/18 of what a resident wave gets of
// the launch, between kBase and 2048.  FP64, 448, 768, 1024 and 2048 each, us:
// 500,000 visibilities and 448 sources 463, 632, 567 and 923, 2,316,722 and 1000
// 3,209, 3,253, 3,311 and 3,538, 9,266,880 and 1000 13,116, 12,850, 12,818 and
// 13,230, of eight channels and 5000 (640 for 448) 468, 464, 459 and 450 ms.  Mixed,
// 448, 640, 1024 and 2048: 1,158,361 and 320 577, 530, 562 and 716, 9,266,880 and
// 1000 9,117, 8,900, 8,831 and 8,958, of eight channels and 5000 (640 on) 315, 311 and
// 309 ms.  Fewer than kBase where those would fill less than kFill % of the
// resident waves (60,000 and 1,500 sources, filling 35, 50 and 70 %: mixed 231 | 255
// | 248 us, FP64 311 | 327 | 286).  A multiple of eight: each wave's first loads then
// start on a line of 128 bytes of every stream (5,000,000 and 256 sources, FP64, 489
// each 2,600 us, 448 and 512 2,157 and 2,184; 1000 sources 7,421 and 6,800).
template <bool kMixed>
int64_t chunk_size(int64_t n_vis, int64_t n_tiles, int64_t capacity) {
  constexpr int64_t kBase = kMixed ? 640 : 448, kFill = kMixed ? 35 : 70, kAlign = 8;
  capacity = std::max<int64_t>(1, capacity);
  const int64_t share = (n_vis * n_tiles + capacity - 1) / capacity;
  const int64_t full = std::min<int64_t>(2048, std::max(kBase, share / 18));
  const int64_t len = std::max(kMinChunk, std::min(full, share * 100 / kFill));
  const int64_t chunks = std::max<int64_t>(1, even_chunks((n_vis + len - 1) / len));
  return std::max(kAlign, ((n_vis + chunks - 1) / chunks + kAlign - 1) / kAlign * kAlign);
}

// Steps of 64 visibilities per wave of k_extract_vp: enough waves to fill the
// chip once, between 2 and 64 steps (a wave ends with two reductions and
// eight atomics per source).  Few chunks rounded up (800 sources, FP64, 11,400 and
// 20,000 visibilities 148 | 107 and 112 | 84 us, mixed form 108 | 101 and 77 | 76).
int64_t vp_steps(int64_t n_vis, int64_t groups, int64_t capacity) {
  const int64_t total = (n_vis + 63) / 64;
  const int64_t fill = (total * groups + capacity - 1) / std::max<int64_t>(1, capacity);
  const int64_t steps = std::min<int64_t>(64, std::max<int64_t>(2, fill));
  const int64_t chunks = std::max<int64_t>(1, even_chunks((total + steps - 1) / steps));
  return std::min<int64_t>(64, std::max<int64_t>(2, (total + chunks - 1) / chunks));
}

// Blocks whose waves cover every (chunk, part): per XCD, the parts of every
// eighth chunk (work_item).
unsigned grid_blocks(int64_t chunks, int64_t parts, int64_t waves) {
  return (unsigned)(kXcd * (((chunks + kXcd - 1) / kXcd * parts + waves - 1) / waves));
}

template <bool kMixed, int NS, bool kUpd>
hipError_t run_vp(ExtractArgs a, const UpdateArgs &u, hipStream_t st) {
  const Sorted &v = a.sv;
  auto kern = k_extract_vp<kMixed, NS, kUpd>;
  constexpr int kW = kVpThreads / 64;
  const int64_t groups = (a.n_src + NS - 1) / NS;
  const int64_t capacity = resident_blocks(kern, kVpThreads) * kW;
  a.chunk = (int32_t)vp_steps(v.n_vis, groups, capacity > 0 ? capacity : 4096);
  const int64_t chunks = (v.n_vis + 64 * (int64_t)a.chunk - 1) / (64 * (int64_t)a.chunk);
  hipLaunchKernelGGL(kern, dim3(grid_blocks(chunks, groups, kW)), dim3(kVpThreads), 0, st, a, v.geo, v.res,
                     reinterpret_cast<const uint64_t *>(v.wt), a.acc.cell, u);
  return hipGetLastError();
}

// FP64: the 1024-entry table, whose blocks are half the size, for 8 to 127 tiles
// where the launch is less than 1.6 rounds of the resident waves.  2048 | 1024
// entries, us: 5,700, 60,000, 200,000 and 240,000 visibilities of 2,000, 3,000,
// 1,000 and 1,000 sources 195 | 156, 472 | 430, 547 | 485 and 557 | 495; at 18,102
// waves (1,158,361 of 448) 840 | 866; 7 tiles (500,000 of 448) 460 | 519, 157 of
// them (2,000 of 10,000) 244 | 270.
template <bool kMixed, int NS, int G, int T>
hipError_t run_tiles(ExtractArgs a, hipStream_t st) {
  const Sorted &v = a.sv;
  auto kern = k_extract<kMixed, NS, G, T>;
  constexpr int kW = waves_per_block<kMixed, T>();
  a.n_tiles = (a.n_src + 64 * NS - 1) / (64 * NS);
  const int64_t capacity = resident_blocks(kern, 64 * kW) * kW;
  a.chunk = (int32_t)chunk_size<kMixed>(v.n_vis, a.n_tiles, capacity);
  a.n_chunks = (v.n_vis + a.chunk - 1) / a.chunk;
  if constexpr (!kMixed && T == 2048)
    if (a.n_tiles >= 8 && a.n_tiles < 128 && a.n_chunks * a.n_tiles * 5 < 8 * capacity) return run_tiles<kMixed, NS, G, 1024>(a, st);
  hipLaunchKernelGGL(kern, dim3(grid_blocks(a.n_chunks, a.n_tiles, kW)), dim3(64 * kW), 0, st, a, v.geo, v.quad, v.res,
                     reinterpret_cast<const uint64_t *>(v.wt), a.acc.cell);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_extract(const ExtractArgs &a, int mixed, hipStream_t st, const UpdateArgs *upd) {
  // the update is fused into the extraction of a single source (a serial
  // refinement): with more, other waves would read the residual meanwhile
  const bool fuse = upd && a.n_src == 1;
  if (fuse) return mixed ? run_vp<true, 1, true>(a, *upd, st) : run_vp<false, 1, true>(a, *upd, st);
  if (upd) {
    hipError_t e = launch_update_sorted(*upd, mixed, st);
    if (e != hipSuccess) return e;
  }
  if (visibilities_on_lanes(a.sv.n_vis, a.n_src, mixed)) {
    const UpdateArgs none{};
    if (a.n_src == 1) return mixed ? run_vp<true, 1, false>(a, none, st) : run_vp<false, 1, false>(a, none, st);
    return mixed ? run_vp<true, 2, false>(a, none, st) : run_vp<false, 2, false>(a, none, st);
  }
  return mixed ? run_tiles<true, kNsMixed, kGroupMixed, 1024>(a, st) : run_tiles<false, kNsF64, kGroupF64, 2048>(a, st);
}

}  // namespace rlf
