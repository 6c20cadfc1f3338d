// The grid-narrowing network: features, BF16 MFMA GEMM, epilogues, loss,
// back-propagation helpers, Adam, and the window boxes.
//
// GEMM: C[M x N] (FP32) = A * B in BF16, both operands contiguous along the
// contraction k (weights, layer inputs and gradients are kept or made
// transposed where a product needs it).  Operand fragments of
// v_mfma_f32_32x32x16_bf16: lane l holds A[l%32][8(l/32)+t] and
// B[8(l/32)+t][l%32] (t = 0..7) and accumulator r of lane l is
// C[8(r/4) + 4(l/32) + r%4][l%32].  grid.z splits K; with more than one split
// each slice writes its partial product to a workspace and a second kernel
// adds the slices in a fixed order, so results do not depend on scheduling.
#include <hip/hip_bf16.h>

#include <algorithm>
#include <cmath>

#include "rlf_internal.h"

namespace rlf {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr float kLogVarMin = -6.9077552789821368f;   // ln(1e-3)
constexpr double kFeatureClip = 4.0;

__device__ __forceinline__ __bf16 to_bf16(float x) { return __float2bfloat16(x); }

// GEMM with both operands contiguous along k: C[M x N] (FP32, row stride
// ldc) = sum_k A[m lda + k] B[n ldb + k].  Block tile 128 x 128, k tile 64,
// four waves each owning a 64 x 64 quarter as 2 x 2
// v_mfma_f32_32x32x16_bf16 tiles.  Both k tiles are staged [row][k] in LDS
// (rows padded to 72 BF16, so the eight lanes of one 16-byte read phase hit
// distinct banks) with 16-byte global loads and LDS stores; the LDS holds two
// k tiles and the registers two more, so the global loads of a tile are
// issued two tiles ahead of its MFMAs, and one barrier per tile separates
// the phases.  Rows beyond M or N and k beyond the slice read as
// zero (K a multiple of 8, lda and ldb multiples of 8).  grid.z splits K in
// slices of kper; with more than one slice each writes its partial product
// to the workspace and k_reduce_split adds the slices in order.
constexpr int kTM = 128, kTN = 128, kTK = 64, kLdT = kTK + 8;

__device__ __forceinline__ void nt_load(bf16x8 (&r)[4], const __bf16 *__restrict__ p, int64_t ld, int r0, int nr,
                                        int k0, int ke) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = threadIdx.x + 256 * j;
    const int row = c >> 3, kc = (c & 7) * 8;
    const int gr = r0 + row, gk = k0 + kc;
    if (gr < nr && gk + 8 <= ke) {
      r[j] = *reinterpret_cast<const bf16x8 *>(p + (int64_t)gr * ld + gk);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) r[j][e] = (gr < nr && gk + e < ke) ? p[(int64_t)gr * ld + gk + e] : to_bf16(0.0f);
    }
  }
}

__device__ __forceinline__ void nt_store(__bf16 *lds, const bf16x8 (&r)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = threadIdx.x + 256 * j;
    *reinterpret_cast<bf16x8 *>(lds + (c >> 3) * kLdT + (c & 7) * 8) = r[j];
  }
}

// The MFMAs of one k tile from LDS into the wave's 2 x 2 accumulator tiles.
__device__ __forceinline__ void nt_mfma(f32x16 (&acc)[2][2], const __bf16 *A, const __bf16 *B, int wm, int wn,
                                        int lane) {
#pragma unroll
  for (int kk = 0; kk < kTK; kk += 16) {
    bf16x8 fa[2], fb[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
      fa[i] = *reinterpret_cast<const bf16x8 *>(A + (wm + i * 32 + (lane & 31)) * kLdT + kk + 8 * (lane >> 5));
#pragma unroll
    for (int j = 0; j < 2; ++j)
      fb[j] = *reinterpret_cast<const bf16x8 *>(B + (wn + j * 32 + (lane & 31)) * kLdT + kk + 8 * (lane >> 5));
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
  }
}

// XCD-aware tile order.  Blocks go to the eight XCDs round-robin by linear
// block index; the tile a block computes is chosen so that each XCD takes a
// contiguous run of tiles in (n tile, m tile, k slice) order, i.e. all the
// n tiles of an m tile (which read the same rows of A) share one XCD's L2.
// Without it the four n tiles of a 512-wide product sat on four XCDs and
// each fetched the same A panel.
__device__ __forceinline__ void nt_tile(int &nt, int &mt, int &z) {
  const int gx = gridDim.x, gy = gridDim.y;
  const int n = gx * gy * (int)gridDim.z;
  const int L = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  const int x = L & 7, r = L >> 3, q = n >> 3, rem = n & 7;
  const int T = x * q + min(x, rem) + r;
  nt = T % gx;
  mt = (T / gx) % gy;
  z = T / (gx * gy);
}

__global__ __launch_bounds__(256) void k_gemm_nt(GemmNTArgs g) {
  __shared__ __attribute__((aligned(16))) __bf16 sa[2][kTM * kLdT];
  __shared__ __attribute__((aligned(16))) __bf16 sb[2][kTN * kLdT];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  int nt, mt, z;
  nt_tile(nt, mt, z);
  const int m0 = mt * kTM, n0 = nt * kTN;
  const int wm = (wid >> 1) * 64, wn = (wid & 1) * 64;
  const int kb = z * g.kper, ke = min(g.K, kb + g.kper);
  const int T = kb < ke ? (ke - kb + kTK - 1) / kTK : 0;      // k tiles of this slice
  f32x16 acc[2][2];
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < 2; ++j)
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  // Two register stages: at the start of step t, LDS half t % 2 holds tile t,
  // stage (t + 1) % 2 tile t + 1 and stage t % 2 tile t + 2 (loads in
  // flight).  After the MFMAs of tile t, tile t + 1 goes to the other LDS
  // half and its stage is reloaded with tile t + 3, so a tile's global loads
  // have two steps of MFMAs to arrive.
  bf16x8 ra0[4], rb0[4], ra1[4], rb1[4];
  auto load = [&](bf16x8 (&ra)[4], bf16x8 (&rb)[4], int t) {
    nt_load(ra, g.a, g.lda, m0, g.M, kb + t * kTK, ke);
    nt_load(rb, g.b, g.ldb, n0, g.N, kb + t * kTK, ke);
  };
  if (T > 0) {
    load(ra0, rb0, 0);
    nt_store(sa[0], ra0);
    nt_store(sb[0], rb0);
  }
  if (T > 1) load(ra1, rb1, 1);
  if (T > 2) load(ra0, rb0, 2);
  __syncthreads();
  for (int t = 0; t < T; t += 2) {
    nt_mfma(acc, sa[0], sb[0], wm, wn, lane);
    if (t + 1 < T) {
      nt_store(sa[1], ra1);
      nt_store(sb[1], rb1);
      if (t + 3 < T) load(ra1, rb1, t + 3);
    }
    __syncthreads();
    if (t + 1 >= T) break;
    nt_mfma(acc, sa[1], sb[1], wm, wn, lane);
    if (t + 2 < T) {
      nt_store(sa[0], ra0);
      nt_store(sb[0], rb0);
      if (t + 4 < T) load(ra0, rb0, t + 4);
    }
    __syncthreads();
  }
  float *outp = gridDim.z > 1 ? g.ws + (int64_t)z * g.M * g.N : g.c;
  const int64_t ld = gridDim.z > 1 ? g.N : g.ldc;
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < 2; ++j)
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + wm + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        const int n = n0 + wn + j * 32 + (lane & 31);
        if (m < g.M && n < g.N) outp[(int64_t)m * ld + n] = acc[i][j][r];
      }
}

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }

__device__ __forceinline__ float gelu_grad(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// Products too small for 128 x 128 tiles to fill the card (512 x 512 is 16 of
// them): one wave per 32 x 32 tile, fragments straight from memory (both
// operands contiguous along k, so a fragment is one 16-byte load per lane),
// 512 k in flight at once, no LDS and no barrier; the bias and GELU of the
// forward pass, or GELU's derivative and the bias gradient's partial sums of
// the backward pass, are applied to the accumulators, and a launch can carry
// a second product beside the first.  Sums run over k in the order of
// k_gemm_nt, the epilogues' in that of k_bias_act and k_gelu_back_colsum, so
// the results are the same bits.  Bound by the latency of the loads.  512
// rows: a forward layer takes 8.0 us (with 128 x 128 tiles, then bias and GELU,
// 12.2 + 4.9), a backward layer, both products, GELU's derivative and the
// transposes, 11.0 us (34).
constexpr int kTileSteps = 16;                   // 16-k steps per register buffer

template <bool kWhole>
__device__ __forceinline__ void tile_load(bf16x8 (&fa)[kTileSteps], bf16x8 (&fb)[kTileSteps], const __bf16 *pa,
                                          const __bf16 *pb, int k0, int ke, int half) {
#pragma unroll
  for (int s = 0; s < kTileSteps; ++s) {
    const int k = k0 + 16 * s;                   // this lane's eight: k + 8 half ...
    if (kWhole || k + 8 * half + 8 <= ke) {
      fa[s] = *reinterpret_cast<const bf16x8 *>(pa + k);
      fb[s] = *reinterpret_cast<const bf16x8 *>(pb + k);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) fa[s][e] = fb[s][e] = to_bf16(0.0f);
    }
  }
}

// One tile's product over k in [kb, ke), ke - kb a multiple of 8.
__device__ __forceinline__ f32x16 tile_product(const TileArgs &g, int m0, int n0, int kb, int ke) {
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const __bf16 *pa = g.a + (int64_t)min(m0 + (lane & 31), g.M - 1) * g.lda + 8 * half;
  const __bf16 *pb = g.b + (int64_t)min(n0 + (lane & 31), g.N - 1) * g.ldb + 8 * half;
  constexpr int kStep = 16 * kTileSteps;
  f32x16 acc;
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  bf16x8 a0[kTileSteps], b0[kTileSteps], a1[kTileSteps], b1[kTileSteps];
  auto load = [&](bf16x8 (&fa)[kTileSteps], bf16x8 (&fb)[kTileSteps], int k0) {
    if (k0 + kStep <= ke)
      tile_load<true>(fa, fb, pa, pb, k0, ke, half);
    else
      tile_load<false>(fa, fb, pa, pb, k0, ke, half);
  };
  auto mul = [&](const bf16x8 (&fa)[kTileSteps], const bf16x8 (&fb)[kTileSteps]) {
#pragma unroll
    for (int s = 0; s < kTileSteps; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s], fb[s], acc, 0, 0, 0);
  };
  load(a0, b0, kb);
  for (int k0 = kb; k0 < ke; k0 += 2 * kStep) {
    if (k0 + kStep < ke) load(a1, b1, k0 + kStep);
    mul(a0, b0);
    if (k0 + 2 * kStep < ke) load(a0, b0, k0 + 2 * kStep);
    if (k0 + kStep < ke) mul(a1, b1);
  }
  return acc;
}

// The tile of block L of n (all of one product) in XCD-aware order, as
// nt_tile: n tiles fastest, then m tiles, then k slices.
__device__ __forceinline__ void tile_of(const TileArgs &g, int L, int n, int &n0, int &m0, int &z) {
  const int gx = (g.N + 31) / 32, gy = (g.M + 31) / 32;
  const int x = L & 7, r = L >> 3, q = n >> 3, rem = n & 7;
  const int T = x * q + min(x, rem) + r;
  n0 = (T % gx) * 32;
  m0 = ((T / gx) % gy) * 32;
  z = T / (gx * gy);
}

__host__ __device__ inline int tile_count(const TileArgs &g) {
  return ((g.N + 31) / 32) * ((g.M + 31) / 32) * g.split;
}

// Element r of lane l's accumulators is row 8(r/4) + 4(l/32) + r%4, column l%32.
template <int kMode>
__global__ __launch_bounds__(64, 1) void k_gemm_tile(TileArgs g1, TileArgs g2) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int n1 = tile_count(g1);
  int m0, n0, z;
  if ((int)blockIdx.x >= n1) {
    const TileArgs &g = g2;
    tile_of(g, blockIdx.x - n1, tile_count(g), n0, m0, z);
    const f32x16 acc = tile_product(g, m0, n0, z * g.kper, min(g.K, (z + 1) * g.kper));
    float *out = g.split > 1 ? g.ws + (int64_t)z * g.M * g.N : g.c;
    const int n = n0 + (lane & 31);
    if (n < g.N)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + 8 * (r >> 2) + 4 * half + (r & 3);
        if (m < g.M) out[(int64_t)m * g.N + n] = acc[r];
      }
    return;
  }
  tile_of(g1, blockIdx.x, n1, n0, m0, z);
  const int n = n0 + (lane & 31);                // N a multiple of 32 here
  if (kMode == kTileForward) {
    const float bias = g1.bias[n];
    const f32x16 acc = tile_product(g1, m0, n0, 0, g1.K);
    bf16x4 hq[4];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = m0 + 8 * (r >> 2) + 4 * half + (r & 3);
      const float v = acc[r] + bias;
      const __bf16 h = to_bf16(gelu(v));
      hq[r >> 2][r & 3] = m < g1.M ? h : to_bf16(0.0f);
      if (m < g1.M) {
        g1.z[(int64_t)m * g1.N + n] = v;
        g1.h[(int64_t)m * g1.N + n] = h;
      }
    }
    if (g1.ht)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = m0 + 8 * q + 4 * half;
        if (m < g1.ldt) *reinterpret_cast<bf16x4 *>(g1.ht + (int64_t)n * g1.ldt + m) = hq[q];
      }
    return;
  }
  float zv[16];
#pragma unroll
  for (int r = 0; r < 16; ++r)
    zv[r] = g1.z[(int64_t)min(m0 + 8 * (r >> 2) + 4 * half + (r & 3), g1.M - 1) * g1.N + n];
  const f32x16 acc = tile_product(g1, m0, n0, 0, g1.K);
  bf16x4 dq[4];
  float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};       // rows g, g + 4, ... in order, g = 0..3
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = m0 + 8 * (r >> 2) + 4 * half + (r & 3);
    const bool in = m < g1.M;
    const float x = in ? acc[r] : 0.0f, gg = in ? gelu_grad(zv[r]) : 0.0f;
    const __bf16 d = to_bf16(x * gg);
    dq[r >> 2][r & 3] = d;
    if (in) g1.dz[(int64_t)m * g1.N + n] = d;
    if (in && g1.c) g1.c[(int64_t)m * g1.N + n] = x;
    const float xo = __shfl_xor(x, 32), go = __shfl_xor(gg, 32);   // the other half's row
    sum[r & 3] = fmaf(half ? xo : x, half ? go : gg, sum[r & 3]);
    sum[r & 3] = fmaf(half ? x : xo, half ? gg : go, sum[r & 3]);
  }
  if (g1.dzt)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int m = m0 + 8 * q + 4 * half;
      if (m < g1.ldt) *reinterpret_cast<bf16x4 *>(g1.dzt + (int64_t)n * g1.ldt + m) = dq[q];
    }
  if (half == 0 && g1.part) g1.part[(int64_t)(m0 / 32) * g1.N + n] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
}

// dst[c][r] = src[r][c] for BF16 matrices [rows x cols], rows of dst ld long
// and zero from `rows` on: 64 x 64 tiles through LDS, four BF16 (8 bytes) per
// global access when the tile is whole
// and the row lengths are multiples of 4, else one element per access.  One
// launch serves several matrices: the blocks run over the tiles of job 0,
// then job 1, ...
struct TransposeBatch {
  int n;
  TransposeJob job[kMaxTransposeJobs];
  int64_t first_tile[kMaxTransposeJobs + 1];   // prefix sums of the jobs' tile counts
  int64_t tiles_x[kMaxTransposeJobs];          // tiles along a job's columns
};

__global__ __launch_bounds__(256) void k_transpose_bf16(TransposeBatch tb) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  __shared__ __bf16 t[64][66];
  const int64_t b = blockIdx.x;
  int jn = 0;
  while (jn + 1 < tb.n && b >= tb.first_tile[jn + 1]) ++jn;
  const TransposeJob &J = tb.job[jn];
  const __bf16 *__restrict__ src = J.src;
  __bf16 *__restrict__ dst = J.dst;
  const int64_t rows = J.rows, cols = J.cols, ld = J.ld;
  const int64_t local = b - tb.first_tile[jn];
  const int64_t r0 = (local / tb.tiles_x[jn]) * 64, c0 = (local % tb.tiles_x[jn]) * 64;
  const bool whole = r0 + 64 <= rows && c0 + 64 <= cols && (cols % 4) == 0 && (ld % 4) == 0 &&
                     ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 7) == 0;
  if (whole) {
    // 64 rows x 16 groups of 4 columns: 4 per thread
    for (int q = threadIdx.x; q < 64 * 16; q += 256) {
      const int i = q >> 4, c4 = (q & 15) * 4;
      const bf16x4 v = *reinterpret_cast<const bf16x4 *>(src + (r0 + i) * cols + c0 + c4);
      for (int e = 0; e < 4; ++e) t[i][c4 + e] = v[e];
    }
    __syncthreads();
    for (int q = threadIdx.x; q < 64 * 16; q += 256) {
      const int j = q >> 4, r4 = (q & 15) * 4;           // output row j = source column c0 + j
      bf16x4 v;
      for (int e = 0; e < 4; ++e) v[e] = t[r4 + e][j];
      *reinterpret_cast<bf16x4 *>(dst + (c0 + j) * ld + r0 + r4) = v;
    }
    return;
  }
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int i = ty; i < 64; i += 4) {
    const int64_t r = r0 + i, c = c0 + tx;
    t[i][tx] = (r < rows && c < cols) ? src[r * cols + c] : to_bf16(0.0f);
  }
  __syncthreads();
  for (int i = ty; i < 64; i += 4) {
    const int64_t c = c0 + i, r = r0 + tx;
    if (c < cols && r < ld) dst[c * ld + r] = t[tx][i];    // zero from rows on
  }
}

// One wave per column: lane j adds slices j, j + 64, ... in order, then the
// lanes are added by a fixed butterfly (the same sum on every run).
__global__ __launch_bounds__(256) void k_colsum_join(const float *part, int slices, int cols, float *db) {
  const int col = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (col >= cols) return;                                   // uniform per wave
  float acc = 0.0f;
  for (int y = lane; y < slices; y += 64) acc += part[(int64_t)y * cols + col];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) acc += __shfl_xor(acc, d);
  if (lane == 0) db[col] = acc;
}

// c[m][n] = sum over slices z = 0, 1, ... of ws[z][m][n], in that order
__global__ __launch_bounds__(256) void k_reduce_split(const float *ws, int split, int M, int N, float *c,
                                                      int64_t ldc) {
  const int64_t total = (int64_t)M * N;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    float acc = ws[i];
    for (int z = 1; z < split; ++z) acc += ws[(int64_t)z * total + i];
    c[(i / N) * ldc + (i % N)] = acc;
  }
}

// z = sum of the slices in order + b, h = GELU(z): k_reduce_split and
// k_bias_act in one pass.
__global__ __launch_bounds__(256) void k_reduce_bias_act(const float *__restrict__ ws, int split,
                                                         const float *__restrict__ b, int64_t rows, int cols,
                                                         float *__restrict__ z, __bf16 *__restrict__ h) {
  const int64_t n = rows * cols;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    float acc = ws[i];
    for (int s = 1; s < split; ++s) acc += ws[(int64_t)s * n + i];
    const float v = acc + b[i % cols];
    z[i] = v;
    h[i] = to_bf16(gelu(v));
  }
}

// z = c + b; h = GELU(z) (BF16) or, for the output layer, y = z (FP32)
__global__ __launch_bounds__(256) void k_bias_act(const float *c, const float *b, int64_t rows, int cols, float *z,
                                                  __bf16 *h, int act) {
  const int64_t n = rows * cols;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float v = c[i] + b[i % cols];
    z[i] = v;
    if (act) h[i] = to_bf16(gelu(v));
  }
}

// The output layer (512 -> 6), whose products are too narrow for the MFMA
// tiles: BF16 operands, FP32 sums in a fixed order.
//   forward:  y[r][j] = sum_k h[r][k] W[k][j] + b[j]; a wave per row, lane l
//             sums k = l, l + 64, ..., then a butterfly over the lanes;
//   gradient: dW[k][j] = sum_r h[r][k] dY_bf16[r][j] and db[j] = sum_r dY[r][j]
//             (3,078 values, the order of W4 and b4 in the parameters) as
//             partial sums over slices of 32 rows, then the slices added by a
//             wave per value in a fixed order;
//   input gradient: dh[r][k] = sum_j dY_bf16[r][j] W[k][j], j = 0..5 in order.
constexpr int kOutW = 512 * 6, kOutWB = 512 * 6 + 6;

__global__ __launch_bounds__(256) void k_out_forward(const __bf16 *__restrict__ h, const __bf16 *__restrict__ w,
                                                     const float *__restrict__ b, int64_t rows, float *y) {
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (r >= rows) return;                                    // whole waves
  float acc[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int k = lane; k < 512; k += 64) {
    const float hv = (float)h[r * 512 + k];
#pragma unroll
    for (int j = 0; j < 6; ++j) acc[j] = fmaf(hv, (float)w[k * 6 + j], acc[j]);
  }
#pragma unroll
  for (int j = 0; j < 6; ++j)
    for (int d = 32; d > 0; d >>= 1) acc[j] += __shfl_xor(acc[j], d);
  if (lane == 0)
#pragma unroll
    for (int j = 0; j < 6; ++j) y[r * 6 + j] = acc[j] + b[j];
}

__global__ __launch_bounds__(256) void k_out_grad_part(const __bf16 *__restrict__ h, const __bf16 *__restrict__ dyb,
                                                       const float *__restrict__ dy, int64_t rows, int64_t per,
                                                       float *part) {
  const int v = blockIdx.x * 256 + threadIdx.x;
  if (v >= kOutWB) return;
  const int64_t r0 = (int64_t)blockIdx.y * per, r1 = min(rows, r0 + per);
  const bool wgt = v < kOutW;
  const int k = wgt ? v / 6 : 0, j = wgt ? v - 6 * (v / 6) : v - kOutW;
  float acc = 0.0f;
  // 32 rows per step, their loads issued together; the sum runs in row order
  for (int64_t rb = r0; rb < r1; rb += 32) {
    float a[32], b[32];
#pragma unroll
    for (int t = 0; t < 32; ++t) {
      const int64_t r = rb + t;
      const bool in = r < r1;
      a[t] = in ? (wgt ? (float)h[r * 512 + k] : 1.0f) : 0.0f;
      b[t] = in ? (wgt ? (float)dyb[r * 6 + j] : dy[r * 6 + j]) : 0.0f;
    }
#pragma unroll
    for (int t = 0; t < 32; ++t) acc = fmaf(a[t], b[t], acc);
  }
  part[(int64_t)blockIdx.y * kOutWB + v] = acc;
}

// One wave per value: lane l adds slices l, l + 64, ... in order, then the
// lanes are added by a fixed butterfly (the same sum on every run).
__global__ __launch_bounds__(256) void k_out_grad_join(const float *part, int slices, float *out) {
  const int v = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (v >= kOutWB) return;                                  // whole waves
  float acc = 0.0f;
  for (int s = lane; s < slices; s += 64) acc += part[(int64_t)s * kOutWB + v];
  for (int d = 32; d > 0; d >>= 1) acc += __shfl_xor(acc, d);
  if (lane == 0) out[v] = acc;
}

__global__ __launch_bounds__(256) void k_out_dh(const __bf16 *__restrict__ dyb, const __bf16 *__restrict__ w,
                                                int64_t rows, float *dh) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < rows * 512; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i >> 9;
    const int k = (int)(i & 511);
    float acc = 0.0f;
#pragma unroll
    for (int j = 0; j < 6; ++j) acc = fmaf((float)dyb[r * 6 + j], (float)w[k * 6 + j], acc);
    dh[i] = acc;
  }
}

// Gaussian negative log-likelihood head: y [n x 6] -> loss (written to
// *loss), dY = dL/dy (FP32 for the bias, BF16 for the products).  The
// log-variance is floored at kLogVarMin (variance 1e-3); below the floor it
// gets no gradient.  Blocks of 1024 threads.  Block 0 forms the loss: thread
// i takes rows i, i + 1024, ... and the terms are added in a fixed order
// (per thread, then a butterfly within each wave, then the waves in order),
// so the loss is the same on every run; it loads kHeadRows rows at a time
// before adding any.  Blocks 1, 2, ... write dY, a row per thread, so that
// the strided loads and stores of a large batch are spread over as many CUs
// (one block's memory pipeline took 17 us for 4096 rows).  Both compute the
// terms by the same expressions (head_terms).
constexpr int kHeadRows = 4;

__device__ __forceinline__ void head_terms(float mu, float s_raw, float tv, float nf, double *lt, float *gm,
                                           float *gs) {
  const float s = fmaxf(s_raw, kLogVarMin);
  const float e = tv - mu;
  const float ie = expf(-s);
  *lt = 0.5 * ((double)s + (double)e * e * ie);
  *gm = -e * ie / nf;
  *gs = s_raw < kLogVarMin ? 0.0f : 0.5f * (1.0f - e * e * ie) / nf;
}

// The loss by one block of 1024 threads (sh: 16 values).
__device__ __forceinline__ void head_loss(const float *__restrict__ y, const float *__restrict__ t, int64_t n,
                                          double *__restrict__ loss, double *sh) {
  const int64_t stride = blockDim.x;
  double acc = 0.0;
  for (int64_t i0 = threadIdx.x; i0 < n; i0 += kHeadRows * stride) {
    float yv[kHeadRows][6], tv[kHeadRows][3];
#pragma unroll
    for (int u = 0; u < kHeadRows; ++u) {
      const int64_t i = i0 + u * stride;
      if (i < n) {
#pragma unroll
        for (int c = 0; c < 6; ++c) yv[u][c] = y[i * 6 + c];
#pragma unroll
        for (int d = 0; d < 3; ++d) tv[u][d] = t[i * 3 + d];
      }
    }
#pragma unroll
    for (int u = 0; u < kHeadRows; ++u) {
      if (i0 + u * stride >= n) break;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        double lt;
        float gm, gs;
        head_terms(yv[u][d], yv[u][3 + d], tv[u][d], (float)n, &lt, &gm, &gs);
        acc += lt;
      }
    }
  }
  for (int d = 32; d > 0; d >>= 1) acc += __shfl_xor(acc, d);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double total = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) total += sh[w];
    *loss = total / (double)n;
  }
}

__global__ __launch_bounds__(1024) void k_head(const float *__restrict__ y, const float *__restrict__ t, int64_t n,
                                               float *__restrict__ dy, __bf16 *__restrict__ dyb,
                                               double *__restrict__ loss) {
  __shared__ double sh[16];
  const int64_t stride = blockDim.x;
  if (blockIdx.x > 0) {
    const int64_t i = (int64_t)(blockIdx.x - 1) * stride + threadIdx.x;
    if (i >= n) return;
    float yv[6], tv[3];
#pragma unroll
    for (int c = 0; c < 6; ++c) yv[c] = y[i * 6 + c];
#pragma unroll
    for (int d = 0; d < 3; ++d) tv[d] = t[i * 3 + d];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      double lt;
      float gm, gs;
      head_terms(yv[d], yv[3 + d], tv[d], (float)n, &lt, &gm, &gs);
      dy[i * 6 + d] = gm;
      dy[i * 6 + 3 + d] = gs;
      dyb[i * 6 + d] = to_bf16(gm);
      dyb[i * 6 + 3 + d] = to_bf16(gs);
    }
    return;
  }
  head_loss(y, t, n, loss, sh);
}

// The output layer of a training step in one launch: a block takes a slice of
// 32 rows through y = h W4 + b4 and the loss gradient, then 128 of the 512
// columns (blockIdx.y) through the slice's part of dW4 and db4, dh = dY W4^T
// and dZ = dh gelu'(Z) with its column sums, with the arithmetic and the order
// of k_out_forward, k_head, k_out_grad_part, k_out_dh and k_gelu_back_colsum.
// (Where the latter's slices are not of 32 rows, dh is written instead of
// their sums, for k_bias_part.)  Bound by latency, a chain of five
// short phases: 512 rows 11.3 us, against 28 us of the five kernels (with all
// 512 columns in one block 20.8 us: sixteen blocks for 256 CUs).
constexpr int kSlice = 32, kHeadCols = 128, kDzLd = kSlice + 2;

__global__ __launch_bounds__(1024) void k_head_slice(HeadArgs a) {
  __shared__ __attribute__((aligned(16))) __bf16 sh[kSlice * 512];
  __shared__ __attribute__((aligned(16))) __bf16 sw[kOutW];
  __shared__ __bf16 sdz[kHeadCols * kDzLd];
  __shared__ float sy[kSlice][6], sdy[kSlice][6], sdyb[kSlice][6], scol[4][kHeadCols];
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * kSlice;
  const int nr = (int)min((int64_t)kSlice, a.rows - r0);
  // last phase: column c, rows g + 4 i with i = 4 up + 0..3
  const int c = t & (kHeadCols - 1), g = (t >> 7) & 3, up = t >> 9;
  const int col = (int)blockIdx.y * kHeadCols + c;
  float zv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) zv[i] = a.z[(r0 + min(g + 16 * up + 4 * i, nr - 1)) * 512 + col];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int e8 = t + 1024 * q;
    bf16x8 v;
    if ((e8 >> 6) < nr)
      v = *reinterpret_cast<const bf16x8 *>(a.h + (r0 + (e8 >> 6)) * 512 + (e8 & 63) * 8);
    else
      for (int e = 0; e < 8; ++e) v[e] = to_bf16(0.0f);
    *reinterpret_cast<bf16x8 *>(sh + e8 * 8) = v;
  }
  if (t < kOutW / 8) *reinterpret_cast<bf16x8 *>(sw + t * 8) = *reinterpret_cast<const bf16x8 *>(a.w + t * 8);
  __syncthreads();
  // the six weights of input k
  auto weights = [&](int k, float (&w)[6]) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const uint32_t u = reinterpret_cast<const uint32_t *>(sw)[k * 3 + q];
      w[2 * q] = __uint_as_float(u << 16);
      w[2 * q + 1] = __uint_as_float(u & 0xffff0000u);
    }
  };
  {                                                         // forward: a wave per two rows
    float acc[2][6] = {};
#pragma unroll
    for (int k = lane; k < 512; k += 64) {
      float w[6];
      weights(k, w);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float hv = (float)sh[(wid + 16 * q) * 512 + k];
#pragma unroll
        for (int j = 0; j < 6; ++j) acc[q][j] = fmaf(hv, w[j], acc[q][j]);
      }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int j = 0; j < 6; ++j) acc[q][j] += __shfl_xor(acc[q][j], d);
    if (lane == 0)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int j = 0; j < 6; ++j) {
          const int r = wid + 16 * q;
          const float yv = acc[q][j] + a.b[j];
          sy[r][j] = yv;
          if (r < nr && blockIdx.y == 0) a.y[(r0 + r) * 6 + j] = yv;
        }
  }
  __syncthreads();
  if (t < kSlice * 3) {                                     // loss gradient
    const int r = t / 3, d = t - 3 * r;
    double lt;
    float gm = 0.0f, gs = 0.0f;
    if (r < nr) head_terms(sy[r][d], sy[r][3 + d], a.target[(r0 + r) * 3 + d], (float)a.rows, &lt, &gm, &gs);
    sdy[r][d] = gm;
    sdy[r][3 + d] = gs;
    sdyb[r][d] = (float)to_bf16(gm);
    sdyb[r][3 + d] = (float)to_bf16(gs);
  }
  __syncthreads();
  float *part = a.out_part + (int64_t)blockIdx.x * kOutWB;
  if (t < kHeadCols * 6) {                                  // dW4 of the slice, and db4
    const int v = (int)blockIdx.y * kHeadCols * 6 + t, k = v / 6, j = v - 6 * k;
    float acc = 0.0f;
#pragma unroll
    for (int r = 0; r < kSlice; ++r) acc = fmaf((float)sh[r * 512 + k], sdyb[r][j], acc);
    part[v] = acc;
  } else if (blockIdx.y == 0 && t < kHeadCols * 6 + 6) {
    float acc = 0.0f;
    for (int r = 0; r < kSlice; ++r) acc = fmaf(1.0f, sdy[r][t - kHeadCols * 6], acc);
    part[kOutW + t - kHeadCols * 6] = acc;
  }
  float w[6], dh[4], gg[4];
  weights(col, w);
#pragma unroll
  for (int i = 0; i < 4; ++i) {                             // dZ
    const int r = g + 16 * up + 4 * i;
    dh[i] = 0.0f;
#pragma unroll
    for (int j = 0; j < 6; ++j) dh[i] = fmaf(sdyb[r][j], w[j], dh[i]);
    gg[i] = r < nr ? gelu_grad(zv[i]) : 0.0f;
    const __bf16 d = to_bf16(dh[i] * gg[i]);
    sdz[c * kDzLd + r] = d;
    if (r < nr) a.dz[(r0 + r) * 512 + col] = d;
    if (r < nr && a.dh) a.dh[(r0 + r) * 512 + col] = dh[i];
  }
  if (up == 0) {                                            // column sums: the upper rows continue the lower ones'
    float acc = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = fmaf(dh[i], gg[i], acc);
    scol[g][c] = acc;
  }
  __syncthreads();
  if (up == 1) {
    float acc = scol[g][c];
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = fmaf(dh[i], gg[i], acc);
    scol[g][c] = acc;
  }
  if (t < kHeadCols * 4) {
    const int k = t >> 2, r = (t & 3) * 8;
    if (r0 + r < a.ldt) {                                   // dZ is zero from row nr on
      bf16x8 v;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = sdz[k * kDzLd + r + e];
      *reinterpret_cast<bf16x8 *>(a.dzt + (int64_t)(blockIdx.y * kHeadCols + k) * a.ldt + r0 + r) = v;
    }
  }
  __syncthreads();
  if (t < kHeadCols && a.part)
    a.part[(int64_t)blockIdx.x * 512 + blockIdx.y * kHeadCols + t] =
        (scol[0][t] + scol[1][t]) + (scol[2][t] + scol[3][t]);
}

// The first step of the bias gradients where their slices are not the tiles'
// 32 rows, one launch for the three hidden layers (blockIdx.z), with the
// arithmetic and the order of k_gelu_back_colsum.  A step of 513 rows takes
// 168 us with it, 209 with the layer's epilogue in kernels of its own for
// such batches.
__global__ __launch_bounds__(256) void k_bias_part(BiasArgs a) {
  __shared__ float sh[4][64];
  const int c = threadIdx.x & 63, rg = threadIdx.x >> 6, l = blockIdx.z;
  const int col = blockIdx.x * 64 + c;
  const float *__restrict__ dh = a.dh[l], *__restrict__ z = a.z[l];
  const int64_t r0 = (int64_t)blockIdx.y * a.per, r1 = min(a.rows, r0 + a.per);
  float acc = 0.0f;
  for (int64_t r = r0 + rg; r < r1; r += 4) acc = fmaf(dh[r * 512 + col], gelu_grad(z[r * 512 + col]), acc);
  sh[rg][c] = acc;
  __syncthreads();
  if (rg == 0) a.part[l][(int64_t)blockIdx.y * 512 + col] = (sh[0][c] + sh[1][c]) + (sh[2][c] + sh[3][c]);
}

// One launch for a step's sums over slices (a wave per value, as
// k_out_grad_join and k_colsum_join) and the loss (block 0).
__global__ __launch_bounds__(1024) void k_join(JoinArgs a) {
  __shared__ double sh[16];
  if (blockIdx.x == 0) {
    head_loss(a.y, a.target, a.rows, a.loss, sh);
    return;
  }
  const int lane = threadIdx.x & 63;
  int v = ((int)blockIdx.x - 1) * 16 + (int)(threadIdx.x >> 6);
  if (v >= kOutWB + 3 * 512) return;                        // whole waves
  const float *p = a.out_part + v;
  float *out = a.gw + v;
  int cols = kOutWB;
  if (v >= kOutWB) {
    v -= kOutWB;
    p = a.part[v >> 9] + (v & 511);
    out = a.db[v >> 9] + (v & 511);
    cols = 512;
  }
  float acc = 0.0f;
  for (int s = lane; s < (cols == 512 ? a.slices : a.out_slices); s += 64) acc += p[(int64_t)s * cols];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) acc += __shfl_xor(acc, d);
  if (lane == 0) *out = acc;
}

// The hidden layers' backward epilogue and the first step of their bias
// gradients in one pass: dZ = dH gelu'(Z) (BF16 copy for the products) over
// a block of 64 columns and a slice of rows, with the slice's column sums
// (four row groups, thread g taking rows g, g + 4, ..., the groups added in
// order) written to part[y][col]; k_colsum_join then adds the slices in
// order, so the sums do not depend on scheduling.
__global__ __launch_bounds__(256) void k_gelu_back_colsum(const float *dh, const float *z, int64_t rows, int cols,
                                                          int64_t per, __bf16 *dzb, float *part) {
  __shared__ float sh[4][64];
  const int col = blockIdx.x * 64 + (threadIdx.x & 63);
  const int rg = threadIdx.x >> 6;
  const int64_t r0 = (int64_t)blockIdx.y * per, r1 = min(rows, r0 + per);
  float acc = 0.0f;
  if (col < cols)
    for (int64_t r = r0 + rg; r < r1; r += 4) {
      const int64_t i = r * cols + col;
      const float v = dh[i] * gelu_grad(z[i]);
      dzb[i] = to_bf16(v);
      acc += v;
    }
  sh[rg][threadIdx.x & 63] = acc;
  __syncthreads();
  if (rg == 0 && col < cols)
    part[(int64_t)blockIdx.y * cols + col] = (sh[0][threadIdx.x] + sh[1][threadIdx.x]) + (sh[2][threadIdx.x] + sh[3][threadIdx.x]);
}

struct AdamConst {
  float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ float adam_value(float w, float g, float &m, float &v, const AdamConst &k) {
  m = fmaf(1.0f - k.b1, g, k.b1 * m);
  v = fmaf(g, (1.0f - k.b2) * g, k.b2 * v);
  return w - k.lr * (m / k.c1) / (sqrtf(v / k.c2) + k.eps);
}

// Adam: the first mt blocks take one 64 x 64 tile of a weight matrix each
// (16 bytes of four arrays per access) and also write its BF16 copy
// transposed through LDS, the others the remaining values one by one.  Bound
// by memory (32 bytes per weight read and written): 25 us for 4.7 million
// weights, 6 TB/s, against 23.4 us without the transposed copy and 7.4 us for
// a pass that made it.
struct AdamTiles {
  int64_t first[AdamMats::kMax + 1];             // first block of a matrix
};

__global__ __launch_bounds__(256) void k_adam(float *w, __bf16 *wb, __bf16 *wbt, const float *g, float *m, float *v,
                                              int64_t n, AdamConst k, AdamMats mats, AdamTiles tiles) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  const int64_t b = blockIdx.x, mt = tiles.first[AdamMats::kMax];
  if (b >= mt) {
    // what lies between and behind the matrices
    for (int64_t i = (b - mt) * 256 + threadIdx.x; i < n; i += ((int64_t)gridDim.x - mt) * 256) {
      int64_t p = i;
#pragma unroll
      for (int j = 0; j < AdamMats::kMax; ++j)
        if (p >= mats.off[j]) p += mats.rows[j] * mats.cols[j];
      float mi = m[p], vi = v[p];
      const float wi = adam_value(w[p], g[p], mi, vi, k);
      m[p] = mi;
      v[p] = vi;
      w[p] = wi;
      wb[p] = to_bf16(wi);
    }
    return;
  }
  __shared__ __bf16 t[64][66];
  int j = 0;
  while (j + 1 < AdamMats::kMax && b >= tiles.first[j + 1]) ++j;
  const int64_t cols = mats.cols[j], rows = mats.rows[j], off = mats.off[j];
  const int64_t local = b - tiles.first[j], tx = cols / 64;
  const int64_t r0 = local / tx * 64, c0 = local % tx * 64;
  const int c4 = (threadIdx.x & 15) * 4, rb = threadIdx.x >> 4;
  float4 wv[4], gv[4], mv[4], vv[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t p = off + (r0 + rb + 16 * q) * cols + c0 + c4;
    wv[q] = *reinterpret_cast<const float4 *>(w + p);
    gv[q] = *reinterpret_cast<const float4 *>(g + p);
    mv[q] = *reinterpret_cast<const float4 *>(m + p);
    vv[q] = *reinterpret_cast<const float4 *>(v + p);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t p = off + (r0 + rb + 16 * q) * cols + c0 + c4;
    float4 x;
    x.x = adam_value(wv[q].x, gv[q].x, mv[q].x, vv[q].x, k);
    x.y = adam_value(wv[q].y, gv[q].y, mv[q].y, vv[q].y, k);
    x.z = adam_value(wv[q].z, gv[q].z, mv[q].z, vv[q].z, k);
    x.w = adam_value(wv[q].w, gv[q].w, mv[q].w, vv[q].w, k);
    const bf16x4 xb = {to_bf16(x.x), to_bf16(x.y), to_bf16(x.z), to_bf16(x.w)};
    *reinterpret_cast<float4 *>(w + p) = x;
    *reinterpret_cast<float4 *>(m + p) = mv[q];
    *reinterpret_cast<float4 *>(v + p) = vv[q];
    *reinterpret_cast<bf16x4 *>(wb + p) = xb;
#pragma unroll
    for (int e = 0; e < 4; ++e) t[rb + 16 * q][c4 + e] = xb[e];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int jc = rb + 16 * q, r4 = (threadIdx.x & 15) * 4;           // output row: column c0 + jc
    bf16x4 x;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = t[r4 + e][jc];
    *reinterpret_cast<bf16x4 *>(wbt + off + (c0 + jc) * rows + r0 + r4) = x;
  }
}

__global__ __launch_bounds__(256) void k_to_bf16(const float *x, __bf16 *y, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = to_bf16(x[i]);
}

// Network input: facet cells inside -32..31 on both axes, Vbar / (S g), g the
// observation's mean spectral factor, clipped to +-kFeatureClip.
__global__ __launch_bounds__(256) void k_features(FeatureArgs a) {
  const int s = a.s0 + (int)blockIdx.x;
  __bf16 *x = a.x + (int64_t)blockIdx.x * 8192;
  for (int i = threadIdx.x; i < 8192; i += blockDim.x) x[i] = to_bf16(0.0f);
  __syncthreads();
  const double inv = 1.0 / (a.src[s].flux * a.spec_norm);
  for (int64_t c = a.offsets[s] + threadIdx.x; c < a.offsets[s + 1]; c += blockDim.x) {
    const int ix = a.ix[c], iy = a.iy[c];
    if (ix < -32 || ix > 31 || iy < -32 || iy > 31) continue;
    const int pos = (iy + 32) * 64 + (ix + 32);
    x[pos] = to_bf16((float)fmin(fmax(a.vre[c] * inv, -kFeatureClip), kFeatureClip));
    x[4096 + pos] = to_bf16((float)fmin(fmax(a.vim[c] * inv, -kFeatureClip), kFeatureClip));
  }
}

// Window boxes from the predictions (decided in FP64 from the FP32 outputs);
// a box covering more than full_frac of the grid becomes the whole grid.
__global__ __launch_bounds__(256) void k_windows(const float *y, int64_t n, double nsigma, int n_e, double step,
                                                 int min_half, double full_frac, int32_t *win) {
  const int c = (n_e - 1) / 2;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    int box[4];
    for (int d = 0; d < 2; ++d) {
      const double mu = (double)y[i * 6 + d];
      const double sd = exp(0.5 * fmax((double)y[i * 6 + 3 + d], (double)kLogVarMin));
      int lo = (int)floor((mu - nsigma * sd) / step + c);
      int hi = (int)ceil((mu + nsigma * sd) / step + c);
      const int mid = (int)rint(mu / step + c);
      lo = min(lo, mid - min_half);
      hi = max(hi, mid + min_half);
      box[2 * d] = min(max(lo, 0), n_e - 1);
      box[2 * d + 1] = min(max(hi, 0), n_e - 1);
    }
    if ((double)(box[1] - box[0] + 1) * (double)(box[3] - box[2] + 1) > full_frac * (double)n_e * (double)n_e) {
      box[0] = box[2] = 0;
      box[1] = box[3] = n_e - 1;
    }
    for (int q = 0; q < 4; ++q) win[i * 4 + q] = box[q];
  }
}

// SplitMix64 (Steele, Lea & Flood, "Fast splittable pseudorandom number
// generators", OOPSLA 2014): the output mix of state seed + k * golden gamma,
// used here as a counter-based generator (value k of stream `seed`).
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t k) {
  uint64_t z = seed + k * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Standard normal number j of stream `seed` by the Box-Muller transform of
// the uniforms u1 = (h(2j+1) >> 11 + 1) 2^-53 in (0, 1] and
// u2 = (h(2j+2) >> 11) 2^-53 in [0, 1), h the counter generator above:
// sqrt(-2 ln u1) cos(2 pi u2), in FP64.
__device__ __forceinline__ double std_normal(uint64_t seed, uint64_t j) {
  const double u1 = ((double)(splitmix64(seed, 2 * j + 1) >> 11) + 1.0) * 0x1.0p-53;
  const double u2 = (double)(splitmix64(seed, 2 * j + 2) >> 11) * 0x1.0p-53;
  return sqrt(-2.0 * log(u1)) * cospi(2.0 * u2);
}

// Training targets drawn around the method's own estimates: row i gets
// (e1_i + kappa s1_i z_{2i}, e2_i + kappa s2_i z_{2i+1}, ln alpha_i) with z
// the normal numbers of stream `seed`; a row whose estimate or spread is not
// finite gets (0, 0, ln alpha_i).
__global__ __launch_bounds__(256) void k_posterior_targets(const double *e1, const double *e2, const double *s1,
                                                           const double *s2, const float *ln_alpha, int64_t n,
                                                           double kappa, uint64_t seed, float *t) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const bool ok = isfinite(e1[i]) && isfinite(e2[i]) && isfinite(s1[i]) && isfinite(s2[i]);
    t[i * 3 + 0] = ok ? (float)(e1[i] + kappa * s1[i] * std_normal(seed, 2 * (uint64_t)i)) : 0.0f;
    t[i * 3 + 1] = ok ? (float)(e2[i] + kappa * s2[i] * std_normal(seed, 2 * (uint64_t)i + 1)) : 0.0f;
    t[i * 3 + 2] = ln_alpha[i];
  }
}

unsigned grid_for(int64_t n) {
  const int64_t b = (n + 255) / 256;
  return (unsigned)(b < 16384 ? (b > 0 ? b : 1) : 16384);
}

}  // namespace

hipError_t launch_bias_act(const float *c, const float *b, int64_t rows, int cols, float *z, __bf16 *h, int act,
                           hipStream_t st) {
  hipLaunchKernelGGL(k_bias_act, dim3(grid_for(rows * cols)), dim3(256), 0, st, c, b, rows, cols, z, h, act);
  return hipGetLastError();
}

hipError_t launch_out_forward(const __bf16 *h, const __bf16 *w, const float *b, int64_t rows, float *y,
                              hipStream_t st) {
  hipLaunchKernelGGL(k_out_forward, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, h, w, b, rows, y);
  return hipGetLastError();
}

hipError_t launch_out_backward(const __bf16 *h, const __bf16 *dyb, const float *dy, int64_t rows, const __bf16 *w,
                               float *gw, float *dh, float *ws, int64_t ws_floats, hipStream_t st) {
  // slices of 32 rows, longer if their partial sums would not fit the workspace
  const int64_t max_slices = ws_floats / kOutWB;
  if (max_slices < 1) return hipErrorInvalidValue;
  const int64_t per = std::max<int64_t>(32, (rows + max_slices - 1) / max_slices);
  const int slices = (int)((rows + per - 1) / per);
  hipLaunchKernelGGL(k_out_grad_part, dim3((kOutWB + 255) / 256, slices), dim3(256), 0, st, h, dyb, dy, rows, per, ws);
  hipLaunchKernelGGL(k_out_grad_join, dim3((kOutWB + 3) / 4), dim3(256), 0, st, ws, slices, gw);
  hipLaunchKernelGGL(k_out_dh, dim3(grid_for(rows * 512)), dim3(256), 0, st, dyb, w, rows, dh);
  return hipGetLastError();
}

hipError_t launch_head(const float *y, const float *t, int64_t n, float *dy, __bf16 *dyb, double *loss,
                       hipStream_t st) {
  hipLaunchKernelGGL(k_head, dim3(1 + (int)((n + 1023) / 1024)), dim3(1024), 0, st, y, t, n, dy, dyb, loss);
  return hipGetLastError();
}

// Row slices of the two-step column sums: at least 32 rows, at most 256
// slices (one block per slice and 64 columns), within the workspace.
void colsum_slices(int64_t rows, int cols, int64_t ws_floats, int64_t *per, int *nsl) {
  const int64_t slices = std::max<int64_t>(1, std::min<int64_t>({256, (rows + 31) / 32, ws_floats / std::max(1, cols)}));
  *per = (rows + slices - 1) / slices;
  *nsl = (int)((rows + *per - 1) / *per);
}

hipError_t launch_gelu_back_colsum(const float *dh, const float *z, int64_t rows, int cols, __bf16 *dzb, float *db,
                                   float *ws, int64_t ws_floats, hipStream_t st) {
  int64_t per;
  int nsl;
  colsum_slices(rows, cols, ws_floats, &per, &nsl);
  hipLaunchKernelGGL(k_gelu_back_colsum, dim3((cols + 63) / 64, nsl), dim3(256), 0, st, dh, z, rows, cols, per, dzb,
                     ws);
  hipLaunchKernelGGL(k_colsum_join, dim3((cols + 3) / 4), dim3(256), 0, st, ws, nsl, cols, db);
  return hipGetLastError();
}

hipError_t launch_gemm_nt(const GemmNTArgs &g, int split_k, hipStream_t st) {
  if (g.K % 8 || g.lda % 8 || g.ldb % 8 || g.kper < 8 || g.kper % 8 || (int64_t)g.kper * std::max(1, split_k) < g.K)
    return hipErrorInvalidValue;
  if (split_k > 1 && (!g.ws || (int64_t)split_k * g.M * g.N > g.ws_floats)) return hipErrorInvalidValue;
  const dim3 grid((g.N + kTN - 1) / kTN, (g.M + kTM - 1) / kTM, split_k > 1 ? split_k : 1);
  hipLaunchKernelGGL(k_gemm_nt, grid, dim3(256), 0, st, g);
  if (split_k > 1 && g.c)
    hipLaunchKernelGGL(k_reduce_split, dim3(grid_for((int64_t)g.M * g.N)), dim3(256), 0, st, g.ws, split_k, g.M, g.N,
                       g.c, g.ldc);
  return hipGetLastError();
}

hipError_t launch_gemm_tile(const TileArgs &first, TileMode mode, const TileArgs *plain, hipStream_t st) {
  const TileArgs *both[2] = {&first, plain};
  for (const TileArgs *g : both) {
    if (!g) continue;
    const bool epi = g == &first;
    if (g->M < 1 || g->N < 1 || g->K < 1 || g->split < 1 || g->K % 8 || g->lda % 8 || g->ldb % 8 ||
        (!epi && (g->kper < 8 || g->kper % 8 || (int64_t)g->kper * g->split < g->K)) ||
        (epi && (g->split != 1 || g->N % 32 ||
                 ((g->ht || g->dzt) && (g->ldt % 8 || g->ldt < g->M || g->ldt >= g->M + 8)))) ||
        (g->split > 1 && !g->ws))
      return hipErrorInvalidValue;
  }
  const TileArgs none{};
  const dim3 grid((unsigned)(tile_count(first) + (plain ? tile_count(*plain) : 0))), block(64);
  if (mode == kTileForward)
    hipLaunchKernelGGL(k_gemm_tile<kTileForward>, grid, block, 0, st, first, plain ? *plain : none);
  else
    hipLaunchKernelGGL(k_gemm_tile<kTileBackward>, grid, block, 0, st, first, plain ? *plain : none);
  if (plain && plain->split > 1)
    hipLaunchKernelGGL(k_reduce_split, dim3(grid_for((int64_t)plain->M * plain->N)), dim3(256), 0, st, plain->ws,
                       plain->split, plain->M, plain->N, plain->c, (int64_t)plain->N);
  return hipGetLastError();
}

hipError_t launch_reduce_bias_act(const float *ws, int split, const float *b, int64_t rows, int cols, float *z,
                                  __bf16 *h, hipStream_t st) {
  hipLaunchKernelGGL(k_reduce_bias_act, dim3(grid_for(rows * cols)), dim3(256), 0, st, ws, split, b, rows, cols, z, h);
  return hipGetLastError();
}

hipError_t launch_head_slice(const HeadArgs &a, hipStream_t st) {
  if (a.rows < 1 || !a.dzt || a.ldt % 8 || a.ldt < a.rows || a.ldt >= a.rows + 8) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_head_slice, dim3((unsigned)((a.rows + kSlice - 1) / kSlice), 512 / kHeadCols), dim3(1024), 0, st,
                     a);
  return hipGetLastError();
}

hipError_t launch_bias_part(const BiasArgs &a, hipStream_t st) {
  if (a.slices < 1 || a.per < 1 || a.per * a.slices < a.rows) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_bias_part, dim3(8, (unsigned)a.slices, 3), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_join(const JoinArgs &a, hipStream_t st) {
  hipLaunchKernelGGL(k_join, dim3(1 + (kOutWB + 3 * 512 + 15) / 16), dim3(1024), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_transpose_bf16(const TransposeJob *jobs, int n_jobs, hipStream_t st) {
  if (n_jobs < 1 || n_jobs > kMaxTransposeJobs) return hipErrorInvalidValue;
  TransposeBatch tb{};
  tb.n = n_jobs;
  tb.first_tile[0] = 0;
  for (int j = 0; j < n_jobs; ++j) {
    // (the cleared columns lie in the tiles of the last rows)
    if (jobs[j].rows < 1 || jobs[j].cols < 1 || jobs[j].ld < jobs[j].rows || jobs[j].ld > (jobs[j].rows + 63) / 64 * 64)
      return hipErrorInvalidValue;
    tb.job[j] = jobs[j];
    tb.tiles_x[j] = (jobs[j].cols + 63) / 64;
    tb.first_tile[j + 1] = tb.first_tile[j] + tb.tiles_x[j] * ((jobs[j].rows + 63) / 64);
  }
  for (int j = n_jobs; j < kMaxTransposeJobs; ++j) tb.first_tile[j + 1] = tb.first_tile[n_jobs];
  hipLaunchKernelGGL(k_transpose_bf16, dim3((unsigned)tb.first_tile[n_jobs]), dim3(256), 0, st, tb);
  return hipGetLastError();
}

hipError_t launch_adam(float *w, __bf16 *wb, __bf16 *wbt, const AdamMats &mats, const float *g, float *m, float *v,
                       int64_t n, float lr, int64_t step, hipStream_t st) {
  const AdamConst k{lr, 0.9f, 0.999f, 1e-8f, (float)(1.0 - std::pow(0.9, (double)step)),
                    (float)(1.0 - std::pow(0.999, (double)step))};
  AdamTiles tiles{};
  int64_t rest = n, end = 0;
  for (int j = 0; j < AdamMats::kMax; ++j) {
    // in order, apart, inside the values, whole tiles, 16-byte accesses
    if (mats.off[j] < end || mats.off[j] % 8 || mats.rows[j] % 64 || mats.cols[j] % 64) return hipErrorInvalidValue;
    const int64_t size = mats.rows[j] * mats.cols[j];
    end = mats.off[j] + size;
    rest -= size;
    tiles.first[j + 1] = tiles.first[j] + size / 4096;
  }
  if (end > n) return hipErrorInvalidValue;
  const int64_t blocks = tiles.first[AdamMats::kMax] + (rest + 255) / 256;
  hipLaunchKernelGGL(k_adam, dim3((unsigned)blocks), dim3(256), 0, st, w, wb, wbt, g, m, v, rest, k, mats, tiles);
  return hipGetLastError();
}

hipError_t launch_to_bf16(const float *x, __bf16 *y, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_to_bf16, dim3(grid_for(n)), dim3(256), 0, st, x, y, n);
  return hipGetLastError();
}

hipError_t launch_features(const FeatureArgs &a, hipStream_t st) {
  hipLaunchKernelGGL(k_features, dim3(a.n_src), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_posterior_targets(const double *e1, const double *e2, const double *s1, const double *s2,
                                   const float *ln_alpha, int64_t n, double kappa, uint64_t seed, float *t,
                                   hipStream_t st) {
  hipLaunchKernelGGL(k_posterior_targets, dim3(grid_for(n)), dim3(256), 0, st, e1, e2, s1, s2, ln_alpha, n, kappa,
                     seed, t);
  return hipGetLastError();
}

hipError_t launch_windows(const float *y, int64_t n, double nsigma, int n_e, double step, int min_half,
                          double full_frac, int32_t *win, hipStream_t st) {
  hipLaunchKernelGGL(k_windows, dim3(grid_for(n)), dim3(256), 0, st, y, n, nsigma, n_e, step, min_half, full_frac,
                     win);
  return hipGetLastError();
}

}  // namespace rlf
