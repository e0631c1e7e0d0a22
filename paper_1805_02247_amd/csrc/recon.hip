// Reconstruction driver support (Sec. 5.2, Sec. 5.3): the vector algebra of L-BFGS over the
// linear modes with FP64 inner products and device-resident scalars, and the binned
// two-point statistics that score a reconstruction (Sec. 4.3).
//
// Inner products: each element product is exact in FP64 (two FP32 factors), the partial
// sums of a fixed grid and the final tree are fixed, so results are bitwise reproducible.
#include "../../include/pmr.h"

#include <mutex>

#include "pmr_internal.h"

namespace pmr {
namespace {

constexpr int TB = 256;
constexpr int DOT_BLOCKS = 1024;  // partial sums per inner product (at most)

// Sum over the block in a fixed tree (pairs 128 apart, then 64, 32, ... 1), on every thread;
// the last six levels stay in the lanes of the first wavefront.
__device__ __forceinline__ double block_sum(double v, double* sh) {
  const int t = threadIdx.x;
  static_assert(TB == 256, "four wavefronts");
  sh[t] = v;
  __syncthreads();
  if (t < 64) {
    double x = (sh[t] + sh[t + 128]) + (sh[t + 64] + sh[t + 192]);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) x += __shfl_down(x, d, 64);
    if (t == 0) sh[0] = x;
  }
  __syncthreads();
  const double r = sh[0];
  __syncthreads();
  return r;
}

int dot_blocks(size_t n) {
  const size_t b = (n + (size_t)TB * 8 - 1) / ((size_t)TB * 8);
  return (int)(b < 1 ? 1 : b > DOT_BLOCKS ? DOT_BLOCKS : b);
}

// The loop bodies below are shared by the kernels with host scalars and the kernels of the
// device-driven optimiser, so both evaluate every element with the same operations: a
// rounded FP32 product then one fused multiply-add, products exact in FP64.

// partial[block] = sum over this block's grid-stride elements of a[i] b[i] (FP64).
__device__ __forceinline__ void dot_partial_body(const float* __restrict__ a,
                                                 const float* __restrict__ b, size_t n,
                                                 double* __restrict__ partial) {
  __shared__ double sh[TB];
  double acc = 0.0;
  const size_t stride = (size_t)gridDim.x * TB;
#pragma unroll 4
  for (size_t i = (size_t)blockIdx.x * TB + threadIdx.x; i < n; i += stride)
    acc += (double)a[i] * (double)b[i];
  const double s = block_sum(acc, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// out = (sum of the partials) / den (den: device scalar, or 1).
__device__ __forceinline__ void dot_final_body(const double* __restrict__ partial, int np,
                                               const double* __restrict__ den,
                                               double* __restrict__ out) {
  __shared__ double sh[TB];
  double acc = 0.0;
  for (int i = threadIdx.x; i < np; i += TB) acc += partial[i];
  const double s = block_sum(acc, sh);
  if (threadIdx.x == 0) out[0] = den ? s / den[0] : s;
}

__device__ __forceinline__ void axpby_body(size_t n, float alpha, const float* a, float beta,
                                           const float* b, float* out) {
  const size_t stride = (size_t)gridDim.x * TB;
  for (size_t i = (size_t)blockIdx.x * TB + threadIdx.x; i < n; i += stride)
    out[i] = __fmaf_rn(beta, b[i], __fmul_rn(alpha, a[i]));
}

__global__ __launch_bounds__(TB) void dot_partial_kernel(const float* __restrict__ a,
                                                         const float* __restrict__ b, size_t n,
                                                         double* __restrict__ partial) {
  dot_partial_body(a, b, n, partial);
}

__global__ __launch_bounds__(TB) void dot_final_kernel(const double* __restrict__ partial, int np,
                                                       const double* __restrict__ den,
                                                       double* __restrict__ out) {
  dot_final_body(partial, np, den, out);
}

// sum of the partials, on every thread of the block, in the fixed tree of dot_final_body.
__device__ __forceinline__ double dot_total(const double* __restrict__ partial, int np) {
  __shared__ double sh[TB];
  double acc = 0.0;
  for (int i = threadIdx.x; i < np; i += TB) acc += partial[i];
  return block_sum(acc, sh);
}

// ---------------------------------------------------------------- two-loop recursion
// d = -H g over a history of `count` pairs in 2 count + 1 launches: each one finishes the inner
// product of the launch before (every workgroup sums its at most DOT_BLOCKS partials, in the
// same tree), updates d with it, and takes the partial sums of the next inner product on
// the values it has just written. An inner product and an update as launches of their own (two
// and one) spent 4-5 us each on as little work: 20 pairs over 2.1e6 elements took 604 us, 363 now.
// The partial sums alternate between two arrays of DOT_BLOCKS.
// Every element and sum is the same operation in the same order as in separate launches.
constexpr int LOOP_U = 4;
enum LoopKind { LOOP_FIRST = 0, LOOP_DOWN = 1, LOOP_UP = 2 };

struct LoopArgs {
  size_t n;
  int kind, j;          // history entry j, newest first
  const float* S;       // [slots][n]
  const float* Y;
  const double* sy;     // per slot
  const double* yy;
  const float* g;
  float* d;
  double* partial;      // [2][DOT_BLOCKS]
  double* alpha;        // per slot
  const float* last;    // nullable: the last launch also takes the partials of last . d
};

// slot(k): the slot of history entry k.
template <class Slot>
__device__ __forceinline__ void loop_body(const LoopArgs& a, int count, Slot slot) {
  const size_t n = a.n;
  const int np = (int)gridDim.x;
  // which of the two arrays the launch reads: launches of one recursion take turns
  const int turn = a.kind == LOOP_FIRST ? 1 : a.kind == LOOP_DOWN ? a.j : 2 * count - 1 - a.j;
  const double* in = a.partial + (size_t)(turn & 1) * DOT_BLOCKS;
  double* out = a.partial + (size_t)((turn + 1) & 1) * DOT_BLOCKS;
  const bool down_end = a.kind == LOOP_DOWN && a.j + 1 == count;
  const bool end = a.kind == LOOP_UP ? a.j == 0 : a.kind == LOOP_FIRST && count == 0;
  const float* x = a.g;
  if (a.kind == LOOP_DOWN) x = a.Y + slot(a.j) * n;
  if (a.kind == LOOP_UP) x = a.S + slot(a.j) * n;
  const float* v = nullptr;  // the other factor of the next inner product
  if (end)
    v = a.last;
  else if (a.kind == LOOP_FIRST)
    v = a.S + slot(0) * n;
  else if (a.kind == LOOP_DOWN)
    v = down_end ? a.Y + slot(a.j) * n : a.S + slot(a.j + 1) * n;
  else
    v = a.Y + slot(a.j - 1) * n;
  // LOOP_U elements per thread in flight; the first ones are asked for before the inner product
  // is finished, which does not need them
  const size_t stride = (size_t)gridDim.x * TB;
  size_t k0 = (size_t)blockIdx.x * TB + threadIdx.x;
  float xr[LOOP_U], dr[LOOP_U], vr[LOOP_U];
  auto load = [&](size_t k) {
#pragma unroll
    for (int u = 0; u < LOOP_U; ++u) {
      const size_t e = k + u * stride;
      const bool in = e < n;
      xr[u] = in ? x[e] : 0.f;
      dr[u] = in && a.kind != LOOP_FIRST ? a.d[e] : 0.f;
      vr[u] = in && v ? v[e] : 0.f;
    }
  };
  load(k0);
  float c = 0.f, gamma = 1.f;
  if (a.kind != LOOP_FIRST) {
    const size_t i = slot(a.j);
    const double q = dot_total(in, np) / a.sy[i];
    if (a.kind == LOOP_DOWN) {  // alpha_i = s_i.q / s_i.y_i; q -= alpha_i y_i
      if (blockIdx.x == 0 && threadIdx.x == 0) a.alpha[i] = q;
      c = (float)(-1.0 * (q - 0.0));
    } else {  // beta = y_i.r / s_i.y_i; r += (alpha_i - beta) s_i
      c = (float)(1.0 * (a.alpha[i] - q));
    }
  }
  if (down_end) {  // r = gamma q, gamma = s.y / y.y of the newest pair
    const size_t i = slot(0);
    gamma = (float)(1.0 * a.sy[i] / a.yy[i]);
  }
  double acc = 0.0;
  while (k0 < n) {
    float xc[LOOP_U], dc[LOOP_U], vc[LOOP_U];
#pragma unroll
    for (int u = 0; u < LOOP_U; ++u) {
      xc[u] = xr[u];
      dc[u] = dr[u];
      vc[u] = vr[u];
    }
    const size_t at = k0;
    k0 += LOOP_U * stride;
    if (k0 < n) load(k0);
#pragma unroll
    for (int u = 0; u < LOOP_U; ++u) {
      const size_t e = at + u * stride;
      if (e < n) {
        float r = a.kind == LOOP_FIRST ? __fmaf_rn(0.f, xc[u], __fmul_rn(1.f, xc[u]))
                                       : __fmaf_rn(c, xc[u], dc[u]);
        if (down_end) r *= gamma;
        if (end) r = __fmaf_rn(0.f, r, __fmul_rn(-1.f, r));
        a.d[e] = r;
        if (v) acc += (double)vc[u] * (double)r;
      }
    }
  }
  if (v) {
    __shared__ double sh[TB];
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
  }
}

struct LoopOrder {
  unsigned char slot[64];
};

__global__ __launch_bounds__(TB) void loop_kernel(LoopArgs a, int count, LoopOrder o) {
  loop_body(a, count, [&](int k) { return (size_t)o.slot[k]; });
}

// ---------------------------------------------------------------- two-loop recursion by its Gram matrix
// Every inner product of the recursion is a combination of those of the s_j and y_j with the
// y_k and g (s_i.q = s_i.g - sum_j alpha_j s_i.y_j, ...), so up to 15 pairs one pass over
// the vectors takes all of them at once, as two 16 x 16 blocks on the FP64 matrix cores
// (products of FP32 values exact, sums in FP64), the scalar recursion runs on them, and one more
// pass combines the vectors. The history is read twice as in the recursion itself, but in
// three launches instead of 2 c + 1, the direction is not written and read back at every
// entry, and it is rounded to FP32 once. An optimiser step over the modes of a 128^3 box with
// 10 pairs: 201 -> 110 us (the Gram pass 48 of them: 28 are the matrix instructions, 36 the reads).
constexpr int GRAM_MAX = 15;       // pairs: with g, the columns of a block
constexpr int GRAM_TB = 512;
constexpr int GRAM_BLOCKS = 256;   // partial Gram matrices at most
constexpr int GRAM_N = 2 * 256;    // [y_j | g].[y_k | g] and s_j.[y_k | g], g in column 15
typedef double gram4 __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));

int gram_blocks(size_t n) {
  const size_t b = (n + 64 * (GRAM_TB / 64) - 1) / (64 * (GRAM_TB / 64));
  return (int)(b < 1 ? 1 : b > GRAM_BLOCKS ? GRAM_BLOCKS : b);
}

// Vector v of block h: y_v (h = 0, also the columns) or s_v, newest first; g at (0, 15).
template <class Slot>
__device__ __forceinline__ const float* gram_vector(const LoopArgs& a, int count, Slot slot,
                                                    int h, int v) {
  if (v < count) return (h ? a.S : a.Y) + slot(v) * a.n;
  return h == 0 && v == GRAM_MAX ? a.g : nullptr;
}

// The same for one or two pairs, on the vector units: the matrix form takes 512 products per
// element whatever the count, of which one pair needs 4 and two need 12. A direction over 2.1e6
// elements took 67 and 68 us with it (38 and 68 as the launches of the recursion), now 33 and 38;
// over 1.7e7 424 and 453 (184 and 329), now 164 and 202. From three pairs on the matrix form is as
// fast or faster (69 against 98, 459 against 472). Bound by reading the vectors.
template <int C, class Slot>
__device__ __forceinline__ void gram_few_body(const LoopArgs& a, Slot slot,
                                              double* __restrict__ out) {
  constexpr int WAVES = GRAM_TB / 64, NE = 2 * C * (C + 1);
  __shared__ double red[WAVES][NE];
  const size_t n = a.n;
  const float* p[2 * C + 1];  // y_j, g, s_j
#pragma unroll
  for (int j = 0; j < C; ++j) {
    p[j] = a.Y + slot(j) * n;
    p[C + 1 + j] = a.S + slot(j) * n;
  }
  p[C] = a.g;
  const bool wide = (n & 3) == 0 && (((uintptr_t)a.S | (uintptr_t)a.Y | (uintptr_t)a.g) & 15) == 0;
  double acc[2][C][C + 1] = {};
  const size_t step = (size_t)gridDim.x * GRAM_TB * 4;
#pragma unroll 2
  for (size_t e = ((size_t)blockIdx.x * GRAM_TB + threadIdx.x) * 4; e < n; e += step) {
    float4v v[2 * C + 1];
#pragma unroll
    for (int q = 0; q <= 2 * C; ++q) {
      if (wide) {
        v[q] = *reinterpret_cast<const float4v*>(p[q] + e);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[q][i] = e + i < n ? p[q][e + i] : 0.f;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < C; ++j)
#pragma unroll
        for (int k = 0; k <= C; ++k) {
          acc[0][j][k] = __builtin_fma((double)v[j][i], (double)v[k][i], acc[0][j][k]);
          acc[1][j][k] = __builtin_fma((double)v[C + 1 + j][i], (double)v[k][i], acc[1][j][k]);
        }
  }
#pragma unroll
  for (int q = 0; q < NE; ++q) {
    double s = acc[q / (C * (C + 1))][q / (C + 1) % C][q % (C + 1)];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) s += __shfl_down(s, d, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][q] = s;
  }
  __syncthreads();
  if (threadIdx.x < NE) {
    const int q = threadIdx.x, h = q / (C * (C + 1)), j = q / (C + 1) % C, k = q % (C + 1);
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < WAVES; ++u) s += red[u][q];
    out[(size_t)blockIdx.x * GRAM_N + h * 256 + j * 16 + (k == C ? GRAM_MAX : k)] = s;
  }
}

// Partial Gram matrices. A wavefront takes 64 elements at a time: lane l holds elements
// 16 q + 4 (l / 16) .. + 3 of vector l % 16 of both blocks, which as operands of
// v_mfma_f64_16x16x4 (A[m][k], B[k][n]: m, n = l % 16, k = l / 16) give the same element to both
// factors whichever k it sits at. C[m][n]: n = l % 16, m = l / 16 + 4 r.
template <class Slot>
__device__ __forceinline__ void gram_body(const LoopArgs& a, int count, Slot slot,
                                          double* __restrict__ out) {
  if (count == 0) return;  // d = -g, which needs none
  if (count == 1) return gram_few_body<1>(a, slot, out);
  if (count == 2) return gram_few_body<2>(a, slot, out);
  constexpr int WAVES = GRAM_TB / 64;
  __shared__ double red[WAVES][GRAM_N / 4];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const size_t n = a.n;
  // rows past the last vector read g and count as zero
  const float* pv[2];
  bool use[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float* p = gram_vector(a, count, slot, h, l & 15);
    use[h] = p != nullptr;
    pv[h] = p ? p : a.g;
  }
  // whole blocks as 16-byte loads where every vector starts on 16 bytes
  const bool wide = (n & 3) == 0 && (((uintptr_t)a.S | (uintptr_t)a.Y | (uintptr_t)a.g) & 15) == 0;
  const size_t step = (size_t)gridDim.x * WAVES * 64;
  size_t e0 = ((size_t)blockIdx.x * WAVES + w) * 64;
  float4v next[2][4];
  auto load = [&](size_t e) {
    const size_t at = e + 4 * (l >> 4);
    if (wide && e + 64 <= n) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          next[h][q] = *reinterpret_cast<const float4v*>(pv[h] + at + 16 * q);
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const size_t k = at + 16 * q + i;
            next[h][q][i] = k < n ? pv[h][k] : 0.f;
          }
    }
  };
  gram4 cy = {0.0, 0.0, 0.0, 0.0}, cs = cy;
  if (e0 < n) load(e0);
  while (e0 < n) {
    float4v cur[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        cur[h][q] = use[h] ? next[h][q] : float4v{0.f, 0.f, 0.f, 0.f};
    e0 += step;
    if (e0 < n) load(e0);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double x = (double)cur[0][q][i], y = (double)cur[1][q][i];
        cy = __builtin_amdgcn_mfma_f64_16x16x4f64(x, x, cy, 0, 0, 0);
        cs = __builtin_amdgcn_mfma_f64_16x16x4f64(y, x, cs, 0, 0, 0);
      }
  }
  // the workgroup's wavefronts in order, a quarter of the entries at a time
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    red[w][l] = cy[r];
    red[w][64 + l] = cs[r];
    __syncthreads();
    for (int t = threadIdx.x; t < GRAM_N / 4; t += GRAM_TB) {
      double s = 0.0;
#pragma unroll
      for (int u = 0; u < WAVES; ++u) s += red[u][t];
      const int lane = t & 63, row = (lane >> 4) + 4 * r, col = lane & 15;
      out[(size_t)blockIdx.x * GRAM_N + (t >> 6) * 256 + row * 16 + col] = s;
    }
    __syncthreads();
  }
}

// d = cg g + sum_j (cy_j y_j + cs_j s_j), rounded once, with the coefficients of -H g from the
// Gram matrix (lane j of the first wavefront follows entry j through both loops); the partial
// sums of last . d in dot_partial_body's order when `last` is given.
template <class Slot>
__device__ __forceinline__ void combine_body(const LoopArgs& a, int count, Slot slot,
                                             const double* __restrict__ G) {
  __shared__ double co[2][16];
  __shared__ double cg_sh;
  const double* GS = G + 256;
  const int t = threadIdx.x;
  if (t < 64) {
    const int j = t < count ? t : 0;
    double alpha = 0.0, delta = 0.0, gamma = 1.0;
    if (count > 0) {
      const size_t i0 = slot(0);
      gamma = a.sy[i0] / a.yy[i0];
      const double sy = a.sy[slot(j)];
      double sq = GS[16 * j + GRAM_MAX];  // s_j.q
      for (int k = 0; k < count; ++k) {              // newest to oldest
        const double ak = __shfl(sq / sy, k, 64);
        if (t == k) alpha = ak;
        sq -= ak * GS[16 * j + k];
      }
      double yr = G[16 * j + GRAM_MAX];  // y_j.r
      for (int k = 0; k < count; ++k) yr -= __shfl(alpha, k, 64) * G[16 * j + k];
      yr *= gamma;
      for (int k = count - 1; k >= 0; --k) {  // oldest to newest
        const double dk = __shfl(alpha - yr / sy, k, 64);
        if (t == k) delta = dk;
        yr += dk * GS[16 * k + j];
      }
    }
    if (t < count) {
      co[0][t] = gamma * alpha;
      co[1][t] = -delta;
    }
    if (t == 0) cg_sh = -gamma;
  }
  __syncthreads();
  const double cg = cg_sh;
  const size_t n = a.n, stride = (size_t)gridDim.x * TB;
  double acc = 0.0;
  constexpr int U = 2;  // elements in flight per thread
  for (size_t k0 = (size_t)blockIdx.x * TB + t; k0 < n; k0 += U * stride) {
    double r[U];
    float gv[U], yv[U][GRAM_MAX], sv[U][GRAM_MAX];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t k = k0 + u * stride;
      const size_t e = k < n ? k : k0;
      gv[u] = a.g[e];
#pragma unroll
      for (int j = 0; j < GRAM_MAX; ++j)
        if (j < count) {
          yv[u][j] = a.Y[slot(j) * n + e];
          sv[u][j] = a.S[slot(j) * n + e];
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      r[u] = cg * (double)gv[u];
#pragma unroll
      for (int j = 0; j < GRAM_MAX; ++j)
        if (j < count) {
          r[u] = __builtin_fma(co[0][j], (double)yv[u][j], r[u]);
          r[u] = __builtin_fma(co[1][j], (double)sv[u][j], r[u]);
        }
      const size_t k = k0 + u * stride;
      if (k < n) {
        const float d = (float)r[u];
        a.d[k] = d;
        if (a.last) acc += (double)gv[u] * (double)d;
      }
    }
  }
  if (a.last) {
    __shared__ double sh[TB];
    const double s = block_sum(acc, sh);
    if (t == 0) a.partial[blockIdx.x] = s;
  }
}

__global__ __launch_bounds__(GRAM_TB) void gram_kernel(LoopArgs a, int count, LoopOrder o,
                                                       double* out) {
  gram_body(a, count, [&](int k) { return (size_t)o.slot[k]; }, out);
}

// total[e] = sum over the partial matrices of entry e, one wavefront per entry (fixed order).
__device__ __forceinline__ void gram_sum_body(const double* __restrict__ part, int blocks,
                                              double* __restrict__ total) {
  const int e = blockIdx.x * (TB / 64) + (threadIdx.x >> 6), l = threadIdx.x & 63;
  double s = 0.0;
  for (int b = l; b < blocks; b += 64) s += part[(size_t)b * GRAM_N + e];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) s += __shfl_down(s, d, 64);
  if (l == 0) total[e] = s;
}

__global__ __launch_bounds__(TB) void gram_sum_kernel(const double* part, int blocks,
                                                      double* total) {
  gram_sum_body(part, blocks, total);
}

__global__ __launch_bounds__(TB) void combine_kernel(LoopArgs a, int count, LoopOrder o,
                                                     const double* G) {
  combine_body(a, count, [&](int k) { return (size_t)o.slot[k]; }, G);
}

// d = -g, the combination without pairs.
__global__ __launch_bounds__(TB) void negate_kernel(size_t n, const float* __restrict__ g,
                                                    float* __restrict__ d) {
  const size_t stride = (size_t)gridDim.x * TB;
  for (size_t i = (size_t)blockIdx.x * TB + threadIdx.x; i < n; i += stride) d[i] = -g[i];
}

// The Gram matrix and its partials in a work buffer, after the partial sums of inner products.
size_t gram_doubles(size_t n) { return (size_t)(gram_blocks(n) + 1) * GRAM_N; }

// out = alpha a + beta b (host scalars; out may alias a or b).
__global__ __launch_bounds__(TB) void axpby_kernel(size_t n, float alpha, const float* a,
                                                   float beta, const float* b, float* out) {
  axpby_body(n, alpha, a, beta, b, out);
}

unsigned stream_grid(size_t n) {
  const size_t b = (n + TB - 1) / TB;
  return (unsigned)(b > 4096 ? 4096 : b < 1 ? 1 : b);
}

// ---------------------------------------------------------------- binned spectra
constexpr int PS_BLOCKS = 1024;  // workgroups at most: partial sums per shell
constexpr int PS_ROWS = 8;       // rows (ix, iy) that share their shells: (+-i, +-j), (+-j, +-i)

// Highest shell that holds a mode: floor(sqrt(3) n / 2).
int top_shell(int n) {
  const long m2 = 3L * (n / 2) * (n / 2);
  long k = 0;
  while ((k + 1) * (k + 1) <= m2) ++k;
  return (int)k;
}

// A wavefront sums the modes of one set of rows at a time: the up to eight rows (+-i, +-j) and
// (+-j, +-i), 0 <= j <= i <= n / 2, have the same shells along kz, so each lane first adds its
// kz of all of them (16 coalesced loads in flight), and one segmented scan over the lanes,
// whose shells ascend with kz, then leaves every shell's sum in the last lane of its run. That
// lane adds it to the wavefront's own LDS slice: one lane per word and instruction, in
// program order, so the sums are bitwise reproducible. The workgroup's slices are added in
// order and go out as partial sums.
// Bound by reading the two spectra once (135 MB at n = 256). One thread per contiguous range
// of modes, each with its slice of a global table, in 8 workgroups of uncoalesced 8-byte
// reads, took 5200 us there, this 34.
template <int CTRL, int RMASK>
__device__ __forceinline__ uint32_t lane_move(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, RMASK, 0xF, RMASK == 0xF);
}
template <int CTRL, int RMASK>
__device__ __forceinline__ double lane_move(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = lane_move<CTRL, RMASK>((uint32_t)u);
  const uint32_t hi = lane_move<CTRL, RMASK>((uint32_t)(u >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

struct ShellSums {
  double v[3];  // |a|^2, |b|^2, Re a conj b
  uint32_t c;   // modes
};

// One step of the segmented scan: keys ascend over the lanes and are never 0 in a lane that a
// move could leave without a source (such a lane reads key 0).
template <int CTRL, int RMASK>
__device__ __forceinline__ void shell_step(ShellSums& s, uint32_t key) {
  const uint32_t k = lane_move<CTRL, RMASK>(key);
  ShellSums o;
#pragma unroll
  for (int q = 0; q < 3; ++q) o.v[q] = lane_move<CTRL, RMASK>(s.v[q]);
  o.c = lane_move<CTRL, RMASK>(s.c);
  if (k == key) {
#pragma unroll
    for (int q = 0; q < 3; ++q) s.v[q] += o.v[q];
    s.c += o.c;
  }
}

__global__ __launch_bounds__(TB) void power_partial_kernel(int n, const float2* __restrict__ a,
                                                           const float2* __restrict__ b,
                                                           int shells, int items, int nbins,
                                                           double* __restrict__ work) {
  extern __shared__ double ps_lds[];  // per wavefront: sums [3][shells], then counts [shells]
  const int lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = n / 2 + 1;
  double* sum = ps_lds + (size_t)w * 3 * shells;
  uint32_t* cnt = reinterpret_cast<uint32_t*>(ps_lds + (size_t)waves * 3 * shells) + w * shells;
  for (int k = lane; k < 3 * shells; k += 64) sum[k] = 0.0;
  for (int k = lane; k < shells; k += 64) cnt[k] = 0u;
  // one chunk of 64 kz of one set of rows at a time, the next one's loads in flight
  struct Chunk {
    float2 a[PS_ROWS], b[PS_ROWS];
    int ij2, z0;
    uint32_t use;
  };
  const int step = gridDim.x * waves;
  int t = blockIdx.x * waves + w, z0 = 0;
  auto load = [&](Chunk& c) {
    // t = i (i + 1) / 2 + j
    int i = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    while (i * (i + 1) / 2 > t) --i;
    const int j = t - i * (i + 1) / 2;
    // distinct indices of +-i and of +-j, and whether (j, i) differs from (i, j)
    const bool mi = i > 0 && 2 * i < n, mj = j > 0 && 2 * j < n, sw = i != j;
    c.ij2 = i * i + j * j;
    c.z0 = z0;
    c.use = 0u;
    const bool in = z0 + lane < h;
#pragma unroll
    for (int r = 0; r < PS_ROWS; ++r) {
      const bool ni = (r & 1) != 0, nj = (r & 2) != 0, flip = (r & 4) != 0;
      const bool use = (!ni || mi) && (!nj || mj) && (!flip || sw);
      c.use |= (use ? 1u : 0u) << r;
      c.a[r] = c.b[r] = make_float2(0.f, 0.f);
      if (use && in) {
        const int ii = ni ? n - i : i, jj = nj ? n - j : j;
        const size_t e = ((size_t)(flip ? jj : ii) * n + (flip ? ii : jj)) * h + z0 + lane;
        c.a[r] = a[e];
        c.b[r] = b[e];
      }
    }
  };
  Chunk next;
  if (t < items) load(next);
  while (t < items) {
    const Chunk c = next;
    z0 += 64;
    if (z0 >= h) {
      z0 = 0;
      t += step;
    }
    if (t < items) load(next);
    const int iz = c.z0 + lane;
    const bool in = iz < h;
    const int m2 = c.ij2 + iz * iz;
    int shell = (int)sqrtf((float)m2);  // floor(sqrt(m2)), corrected to the exact integer
    shell += (shell + 1) * (shell + 1) <= m2 ? 1 : 0;
    shell -= shell * shell > m2 ? 1 : 0;
    const double wz = (iz == 0 || 2 * iz == n) ? 1.0 : 2.0;
    ShellSums s{{0.0, 0.0, 0.0}, 0u};
    if (in && m2 > 0) {
#pragma unroll
      for (int r = 0; r < PS_ROWS; ++r)
        if ((c.use >> r) & 1u) {
          const float2 av = c.a[r], bv = c.b[r];
          s.v[0] += wz * ((double)av.x * av.x + (double)av.y * av.y);
          s.v[1] += wz * ((double)bv.x * bv.x + (double)bv.y * bv.y);
          s.v[2] += wz * ((double)av.x * bv.x + (double)av.y * bv.y);
          s.c += (uint32_t)wz;
        }
    }
    // shell 0 holds the excluded mode only; lanes past the row get keys of their own
    const uint32_t key = in ? (uint32_t)shell + 1u : 0x40000000u + (uint32_t)lane;
    shell_step<0x111, 0xF>(s, key);  // row_shr 1, 2, 4, 8
    shell_step<0x112, 0xF>(s, key);
    shell_step<0x114, 0xF>(s, key);
    shell_step<0x118, 0xF>(s, key);
    shell_step<0x142, 0xA>(s, key);  // row_bcast 15, 31
    shell_step<0x143, 0xC>(s, key);
    const uint32_t up = (uint32_t)__shfl_down((int)key, 1, 64);
    if (in && (lane == 63 || up != key) && shell > 0 && shell < shells) {
#pragma unroll
      for (int q = 0; q < 3; ++q) sum[q * shells + shell] += s.v[q];
      cnt[shell] += s.c;
    }
  }
  __syncthreads();
  const uint32_t* c0 = reinterpret_cast<const uint32_t*>(ps_lds + (size_t)waves * 3 * shells);
  for (int k = threadIdx.x; k < shells; k += blockDim.x) {
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int u = 0; u < waves; ++u) {
      v[0] += (double)c0[u * shells + k];
#pragma unroll
      for (int q = 0; q < 3; ++q) v[q + 1] += ps_lds[((size_t)u * 3 + q) * shells + k];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) work[((size_t)q * nbins + k) * PS_BLOCKS + blockIdx.x] = v[q];
  }
}

// out[q][bin] = sum over the workgroups of work[q][bin][block] (fixed tree); spectra normalised
// by the mode count and L^3 / n^6. Shells past the last that holds a mode are zero.
__global__ __launch_bounds__(TB) void power_reduce_kernel(const double* __restrict__ work,
                                                          int nbins, int shells, int blocks,
                                                          double norm, double* __restrict__ out) {
  __shared__ double sh[TB];
  const int bin = blockIdx.x;
  double s[4];
  for (int q = 0; q < 4; ++q) {
    double acc = 0.0;
    const double* src = work + ((size_t)q * nbins + bin) * PS_BLOCKS;
    if (bin < shells)
      for (int t = threadIdx.x; t < blocks; t += TB) acc += src[t];
    s[q] = block_sum(acc, sh);
  }
  if (threadIdx.x == 0) {
    const double c = s[0];
    out[bin] = c;
    for (int q = 1; q < 4; ++q) out[(size_t)q * nbins + bin] = c > 0 ? s[q] * norm / c : 0.0;
  }
}

}  // namespace

// Partial sums of the three inner products of a candidate pair (the recursion uses two arrays),
// then the Gram matrices.
size_t vec_work_doubles(size_t n) { return (size_t)3 * DOT_BLOCKS + 64 + gram_doubles(n); }

void launch_vec_dot(size_t n, const float* a, const float* b, const double* den, double* out,
                    double* work, hipStream_t s) {
  const int nb = dot_blocks(n);
  dot_partial_kernel<<<nb, TB, 0, s>>>(a, b, n, work);
  dot_final_kernel<<<1, TB, 0, s>>>(work, nb, den, out);
}

void launch_vec_axpby(size_t n, float alpha, const float* a, float beta, const float* b,
                      float* out, hipStream_t s) {
  axpby_kernel<<<stream_grid(n), TB, 0, s>>>(n, alpha, a, beta, b, out);
}

// d = -H g by the two-loop recursion. order[0..count): history slots, newest first. sy, yy:
// s.y and y.y per slot (device). work: two arrays of partial sums; gram: gram_doubles(n); scal:
// alpha per slot. The Gram form takes any count it has room for, in buffers of up to one slot
// more than that: the same choice as the device-driven optimiser's (by its history length), so
// that both drivers' directions agree bit for bit.
void launch_lbfgs_direction(size_t n, int m, int count, const int* order, const float* S,
                            const float* Y, const double* sy, const double* yy, const float* g,
                            float* d, double* work, double* gram, double* scal, hipStream_t s) {
  const int nb = dot_blocks(n);
  LoopArgs a{n, LOOP_FIRST, 0, S, Y, sy, yy, g, d, work, scal, nullptr};
  LoopOrder o{};
  for (int j = 0; j < count; ++j) o.slot[j] = (unsigned char)order[j];
  if (count <= GRAM_MAX && m <= GRAM_MAX + 1) {
    if (count == 0) {
      negate_kernel<<<stream_grid(n), TB, 0, s>>>(n, g, d);
      return;
    }
    const int gb = gram_blocks(n);
    double* total = gram + (size_t)gb * GRAM_N;
    gram_kernel<<<gb, GRAM_TB, 0, s>>>(a, count, o, gram);
    gram_sum_kernel<<<GRAM_N / (TB / 64), TB, 0, s>>>(gram, gb, total);
    combine_kernel<<<nb, TB, 0, s>>>(a, count, o, total);
    return;
  }
  loop_kernel<<<nb, TB, 0, s>>>(a, count, o);
  a.kind = LOOP_DOWN;
  for (a.j = 0; a.j < count; ++a.j) loop_kernel<<<nb, TB, 0, s>>>(a, count, o);  // newest first
  a.kind = LOOP_UP;
  for (a.j = count - 1; a.j >= 0; --a.j) loop_kernel<<<nb, TB, 0, s>>>(a, count, o);
}

// ---------------------------------------------------------------- device-driven L-BFGS
// Every kernel below reads the optimiser state first and returns at once (all threads
// alike) unless the state is in the phase it belongs to; so a fixed sequence of launches --
// capturable as a graph -- performs whichever branch the device-side tests chose.
namespace {

enum Gate {
  G_RUN = 0,   // the stage is running
  G_ACC = 1,   // the last trial was accepted (the pair and the move to x_t)
  G_DIR = 2,   // accepted and still running (the next direction)
  G_RESET = 3  // ... and that direction was not a descent direction
};
// A kernel with jc >= 0 (history entry jc) runs only while jc < state.count.

__device__ __forceinline__ bool gate_open(const pmr_lbfgs_state* st, int gate, int jc) {
  bool on;
  if (gate == G_RUN)
    on = st->status == PMR_LBFGS_RUNNING;
  else if (gate == G_ACC)
    on = st->accepted != 0;
  else if (gate == G_DIR)
    on = st->accepted != 0 && st->status == PMR_LBFGS_RUNNING;
  else
    on = st->accepted != 0 && st->status == PMR_LBFGS_RUNNING && st->reset != 0;
  return on && (jc < 0 || jc < st->count);
}

__device__ __forceinline__ double* f_hist(pmr_lbfgs_state* st) {
  return reinterpret_cast<double*>(st + 1);
}
__device__ __forceinline__ long long* clock_hist(pmr_lbfgs_state* st) {
  return reinterpret_cast<long long*>(f_hist(st) + st->p.max_iter + 1);
}

__global__ __launch_bounds__(TB) void lb_dot_partial_kernel(const pmr_lbfgs_state* st, int gate,
                                                            const float* A, const float* B,
                                                            size_t n, double* partial) {
  if (!gate_open(st, gate, -1)) return;
  dot_partial_body(A, B, n, partial);
}

// One launch of the recursion over the device-held history (entry j >= count: nothing).
__global__ __launch_bounds__(TB) void lb_loop_kernel(const pmr_lbfgs_state* st, LoopArgs a) {
  if (!gate_open(st, G_DIR, a.kind == LOOP_FIRST ? -1 : a.j)) return;
  loop_body(a, st->count, [&](int k) { return (size_t)st->order[k]; });
}

// The Gram form of the same, for the newest GRAM_MAX pairs: more are held only where the update's
// m is not the state's, and then the form still keeps to its blocks.
__device__ __forceinline__ int gram_count(const pmr_lbfgs_state* st) {
  return st->count < GRAM_MAX ? st->count : GRAM_MAX;
}
__global__ __launch_bounds__(GRAM_TB) void lb_gram_kernel(const pmr_lbfgs_state* st, LoopArgs a,
                                                          double* out) {
  if (!gate_open(st, G_DIR, -1)) return;
  gram_body(a, gram_count(st), [&](int k) { return (size_t)st->order[k]; }, out);
}
__global__ __launch_bounds__(TB) void lb_gram_sum_kernel(const pmr_lbfgs_state* st,
                                                         const double* part, int blocks,
                                                         double* total) {
  if (!gate_open(st, G_DIR, 0)) return;
  gram_sum_body(part, blocks, total);
}
__global__ __launch_bounds__(TB) void lb_combine_kernel(const pmr_lbfgs_state* st, LoopArgs a,
                                                        const double* G) {
  if (!gate_open(st, G_DIR, -1)) return;
  combine_body(a, gram_count(st), [&](int k) { return (size_t)st->order[k]; }, G);
}

// The candidate pair of an accepted trial, s = xt - x and y = gt - g, into its slot, with the
// partial sums of s.y, y.y and s.s.
__global__ __launch_bounds__(TB) void lb_pair_kernel(const pmr_lbfgs_state* st, size_t n,
                                                     const float* xt, const float* x,
                                                     const float* gt, const float* g, float* S,
                                                     float* Y, double* partial) {
  if (!gate_open(st, G_ACC, -1)) return;
  __shared__ double sh[TB];
  float* sv = S + (size_t)st->slot * n;
  float* yv = Y + (size_t)st->slot * n;
  double acc[3] = {0.0, 0.0, 0.0};
  const size_t stride = (size_t)gridDim.x * TB;
  for (size_t i = (size_t)blockIdx.x * TB + threadIdx.x; i < n; i += stride) {
    const float sx = __fmaf_rn(-1.f, x[i], __fmul_rn(1.f, xt[i]));
    const float yx = __fmaf_rn(-1.f, g[i], __fmul_rn(1.f, gt[i]));
    sv[i] = sx;
    yv[i] = yx;
    acc[0] += (double)sx * (double)yx;
    acc[1] += (double)yx * (double)yx;
    acc[2] += (double)sx * (double)sx;
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const double t = block_sum(acc[q], sh);
    if (threadIdx.x == 0) partial[(size_t)q * DOT_BLOCKS + blockIdx.x] = t;
  }
}

// The move to the accepted trial, x = xt and g = gt, with the partial sums of g.g.
__global__ __launch_bounds__(TB) void lb_move_kernel(const pmr_lbfgs_state* st, size_t n,
                                                     const float* xt, float* x, const float* gt,
                                                     float* g, double* partial) {
  if (!gate_open(st, G_ACC, -1)) return;
  __shared__ double sh[TB];
  double acc = 0.0;
  const size_t stride = (size_t)gridDim.x * TB;
  for (size_t i = (size_t)blockIdx.x * TB + threadIdx.x; i < n; i += stride) {
    x[i] = __fmaf_rn(0.f, xt[i], __fmul_rn(1.f, xt[i]));
    const float v = __fmaf_rn(0.f, gt[i], __fmul_rn(1.f, gt[i]));
    g[i] = v;
    acc += (double)v * (double)v;
  }
  const double t = block_sum(acc, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// out = alpha a + beta b
__global__ __launch_bounds__(TB) void lb_axpby_kernel(const pmr_lbfgs_state* st, int gate,
                                                      size_t n, float alpha, const float* a,
                                                      float beta, const float* b, float* out) {
  if (!gate_open(st, gate, -1)) return;
  axpby_body(n, alpha, a, beta, b, out);
}

// xt = x + t d
__global__ __launch_bounds__(TB) void lb_trial_kernel(const pmr_lbfgs_state* st, size_t n,
                                                      const float* x, const float* d, float* xt) {
  if (st->status != PMR_LBFGS_RUNNING) return;
  axpby_body(n, 1.f, x, (float)st->t, d, xt);
}

__global__ void lb_init_kernel(pmr_lbfgs_state* st, pmr_lbfgs_params p, const double* loss,
                               long long clock_khz) {
  st->p = p;
  st->clock_khz = clock_khz;
  st->f = loss[0];
  st->ft = st->f;
  st->t = 0.0;
  st->gd = st->gg = st->rel = st->ss = st->beta = 0.0;
  st->status = PMR_LBFGS_RUNNING;
  st->iters = 0;
  st->evals = 1;
  st->count = 0;
  st->halvings = 0;
  st->probe = 1;
  st->accepted = 1;  // opens the direction kernels that follow
  st->slot = 0;
  st->reset = 0;
  f_hist(st)[0] = st->f;
  clock_hist(st)[0] = wall_clock64();
}

// g.g from its partials; a zero gradient ends the stage
__global__ __launch_bounds__(TB) void lb_gg_kernel(pmr_lbfgs_state* st, const double* partial,
                                                   int np) {
  if (!gate_open(st, G_DIR, -1)) return;
  const double gg = dot_total(partial, np);
  if (threadIdx.x != 0) return;
  st->gg = gg;
  if (gg == 0.0) st->status = PMR_LBFGS_STATIONARY;
}

// g.d from its partials; not a descent direction: clear the history, d = -g follows. Then the
// first trial step of the search.
__global__ __launch_bounds__(TB) void lb_gd_kernel(pmr_lbfgs_state* st, const double* partial,
                                                   int np) {
  if (!gate_open(st, G_DIR, -1)) return;
  const double gd = dot_total(partial, np);
  if (threadIdx.x != 0) return;
  if (gd >= 0.0) {
    st->count = 0;
    st->reset = 1;
    st->gd = -st->gg;
  } else {
    st->reset = 0;
    st->gd = gd;
  }
  st->probe = st->count == 0;
  st->t = st->probe ? __ddiv_rn(1.0, __dsqrt_rn(st->gg)) : 1.0;
  st->halvings = 0;
}

// Armijo test of the trial; on rejection halve t, on acceptance pick the candidate slot
__global__ void lb_test_kernel(pmr_lbfgs_state* st, const double* loss) {
  if (st->status != PMR_LBFGS_RUNNING) {
    st->accepted = 0;
    return;
  }
  st->evals += 1;
  st->ft = loss[0];
  const double bound = __dadd_rn(st->f, __dmul_rn(__dmul_rn(st->p.c1, st->t), st->gd));
  st->accepted = st->ft <= bound;
  if (!st->accepted) {
    st->t *= 0.5;
    if (++st->halvings > st->p.max_halvings) st->status = PMR_LBFGS_LINE_SEARCH;
    return;
  }
  for (int k = 0; k <= st->p.m; ++k) {
    bool used = false;
    for (int j = 0; j < st->count; ++j) used = used || st->order[j] == k;
    if (!used) {
      st->slot = k;
      break;
    }
  }
}

// inner products of the candidate pair, curvature test, history update and the stopping rules
__global__ __launch_bounds__(TB) void lb_accept_kernel(pmr_lbfgs_state* st,
                                                       const double* partial, int np, double* sy,
                                                       double* yy) {
  if (!gate_open(st, G_ACC, -1)) return;
  const double p[3] = {dot_total(partial, np), dot_total(partial + DOT_BLOCKS, np),
                       dot_total(partial + 2 * DOT_BLOCKS, np)};
  if (threadIdx.x != 0) return;
  const int i = st->slot;
  sy[i] = p[0];
  yy[i] = p[1];
  st->ss = p[2];
  if (sy[i] > __dmul_rn(st->p.curvature_eps, __dsqrt_rn(__dmul_rn(yy[i], st->ss)))) {
    const int keep = st->count < st->p.m ? st->count : st->p.m - 1;
    for (int k = keep; k > 0; --k) st->order[k] = st->order[k - 1];
    st->order[0] = i;
    st->count = keep + 1;
  }
  st->rel = st->f != 0.0 ? __ddiv_rn(__dsub_rn(st->f, st->ft), fabs(st->f)) : 0.0;
  st->f = st->ft;
  st->iters += 1;
  f_hist(st)[st->iters] = st->f;
  clock_hist(st)[st->iters] = wall_clock64();
  if (st->f <= st->p.stop_below)
    st->status = PMR_LBFGS_TARGET;
  else if (st->rel < st->p.rel_tol && !st->probe)
    st->status = PMR_LBFGS_CONVERGED;
  else if (st->iters >= st->p.max_iter)
    st->status = PMR_LBFGS_MAX_ITER;
}

}  // namespace

// The next direction at x (g), whose g.g partials are at the start of `work`: the
// zero-gradient test, the two-loop recursion over the device-held history, the descent test
// with its fallback d = -g, and the first step.
void lb_direction(pmr_lbfgs_state* st, size_t n, int m, const float* g, float* d, const float* S,
                  const float* Y, const double* sy, const double* yy, double* work,
                  hipStream_t s) {
  const int nb = dot_blocks(n);
  lb_gg_kernel<<<1, TB, 0, s>>>(st, work, nb);
  LoopArgs a{n, LOOP_FIRST, 0, S, Y, sy, yy, g, d, work, st->alpha, g};
  if (m <= GRAM_MAX) {
    const int gb = gram_blocks(n);
    double* gram = work + 3 * DOT_BLOCKS + 64;
    double* total = gram + (size_t)gb * GRAM_N;
    lb_gram_kernel<<<gb, GRAM_TB, 0, s>>>(st, a, gram);
    lb_gram_sum_kernel<<<GRAM_N / (TB / 64), TB, 0, s>>>(st, gram, gb, total);
    lb_combine_kernel<<<nb, TB, 0, s>>>(st, a, total);
  } else {
    lb_loop_kernel<<<nb, TB, 0, s>>>(st, a);
    a.kind = LOOP_DOWN;
    for (a.j = 0; a.j < m; ++a.j) lb_loop_kernel<<<nb, TB, 0, s>>>(st, a);  // newest to oldest
    a.kind = LOOP_UP;
    for (a.j = m - 1; a.j >= 0; --a.j) lb_loop_kernel<<<nb, TB, 0, s>>>(st, a);  // to newest
  }
  // (either way the partials of g.d are in the first array: after 2 count + 1 launches that ran,
  // or from the combination)
  lb_gd_kernel<<<1, TB, 0, s>>>(st, work, nb);
  lb_axpby_kernel<<<stream_grid(n), TB, 0, s>>>(st, G_RESET, n, -1.f, g, 0.f, g, d);
}

void launch_lbfgs_init(size_t n, const pmr_lbfgs_params& p, pmr_lbfgs_state* st,
                       const double* loss, const float* g, float* d, const float* S,
                       const float* Y, const double* sy, const double* yy, double* work,
                       long long clock_khz, hipStream_t s) {
  lb_init_kernel<<<1, 1, 0, s>>>(st, p, loss, clock_khz);
  lb_dot_partial_kernel<<<dot_blocks(n), TB, 0, s>>>(st, G_DIR, g, g, n, work);
  lb_direction(st, n, p.m, g, d, S, Y, sy, yy, work, s);
}

void launch_lbfgs_trial(size_t n, const pmr_lbfgs_state* st, const float* x, const float* d,
                        float* xt, hipStream_t s) {
  lb_trial_kernel<<<stream_grid(n), TB, 0, s>>>(st, n, x, d, xt);
}

void launch_lbfgs_update(size_t n, int m, pmr_lbfgs_state* st, const double* loss, float* x,
                         float* g, const float* xt, const float* gt, float* d, float* S,
                         float* Y, double* sy, double* yy, double* work, hipStream_t s) {
  const int nb = dot_blocks(n);
  lb_test_kernel<<<1, 1, 0, s>>>(st, loss);
  lb_pair_kernel<<<nb, TB, 0, s>>>(st, n, xt, x, gt, g, S, Y, work);
  lb_accept_kernel<<<1, TB, 0, s>>>(st, work, nb, sy, yy);
  lb_move_kernel<<<nb, TB, 0, s>>>(st, n, xt, x, gt, g, work);
  lb_direction(st, n, m, g, d, S, Y, sy, yy, work, s);
}

size_t power_work_doubles(int nbins) { return (size_t)4 * nbins * PS_BLOCKS; }

void launch_power_bins(int n, double box, const float2* a, const float2* b, int nbins,
                       double* out, double* work, hipStream_t s) {
  const int top = top_shell(n) + 1, shells = nbins < top ? nbins : top;
  const int items = (n / 2 + 1) * (n / 2 + 2) / 2;
  // 28 bytes of LDS per shell and wavefront, at most 64 KB (two wavefronts at n = 1024)
  const int waves = shells * 28 * 4 <= 64 * 1024 ? 4 : 2;
  const int need = (items + waves - 1) / waves, blocks = need < PS_BLOCKS ? need : PS_BLOCKS;
  power_partial_kernel<<<blocks, 64 * waves, (size_t)waves * shells * 28, s>>>(
      n, a, b, shells, items, nbins, work);
  const double norm = box * box * box / ((double)n * n * n * (double)n * n * n);
  power_reduce_kernel<<<nbins, TB, 0, s>>>(work, nbins, shells, blocks, norm, out);
}

}  // namespace pmr

// ---------------------------------------------------------------- fixed scratch
// The scratch of pmr_lbfgs_direction_noalloc: the two arrays of partial sums, the two-loop
// scalars (alpha per slot: at most 64) and the Gram matrices, 1.07 MB. One copy per GPU, held until
// the process ends; every call on a GPU shares it, so calls that overlap on one GPU (several
// streams or threads) race.
constexpr int NOALLOC_MAX_M = 64;
constexpr size_t NOALLOC_DOUBLES = (size_t)2 * pmr::DOT_BLOCKS + NOALLOC_MAX_M +
                                   (size_t)(pmr::GRAM_BLOCKS + 1) * pmr::GRAM_N;
static __device__ __align__(256) double scratch[NOALLOC_DOUBLES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_dev[kMaxDevices] = {};  // device address of `scratch` on each GPU

// Device address of this GPU's copy of `scratch` (the GPU that runs `stream`), taken once per
// device with that device current. In host code the array's name is only a stand-in for
// the symbol, so kernels get this address instead.
int scratch_of(hipStream_t stream, double** out) {
  int cur = 0;
  if (hipGetDevice(&cur) != hipSuccess) return PMR_E_HIP;
  int dev = cur;
  if (stream && hipStreamGetDevice(stream, &dev) != hipSuccess) return PMR_E_HIP;
  if (dev < 0 || dev >= kMaxDevices) return PMR_E_SHAPE;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    if (dev != cur && hipSetDevice(dev) != hipSuccess) return PMR_E_HIP;
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (dev != cur) (void)hipSetDevice(cur);
    if (e != hipSuccess || !p) return PMR_E_HIP;
    g_scratch_dev[dev] = static_cast<double*>(p);
  }
  *out = g_scratch_dev[dev];
  return PMR_OK;
}
}  // namespace

// ---------------------------------------------------------------- C ABI
using namespace pmr;

extern "C" {

size_t pmr_vec_work_bytes(size_t n, int m) {
  if (m < 0) return 0;
  return (vec_work_doubles(n) + (size_t)m + 8) * sizeof(double);
}

int pmr_vec_dot(size_t n, const float* a, const float* b, double* out, void* work, void* stream) {
  if (!a || !b || !out || !work || n == 0) return PMR_E_INVALID;
  launch_vec_dot(n, a, b, nullptr, out, (double*)work, (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? PMR_OK : PMR_E_HIP;
}

int pmr_vec_axpby(size_t n, double alpha, const float* a, double beta, const float* b,
                  float* out, void* stream) {
  if (!a || !b || !out || n == 0) return PMR_E_INVALID;
  launch_vec_axpby(n, (float)alpha, a, (float)beta, b, out, (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? PMR_OK : PMR_E_HIP;
}

int pmr_lbfgs_direction(size_t n, int m, int count, const int* order, const float* S,
                        const float* Y, const double* sy, const double* yy, const float* g,
                        float* d, void* work, void* stream) {
  if (!g || !d || !work || n == 0 || g == d || m < 1 || m > 64 || count < 0 || count > m)
    return PMR_E_INVALID;
  if (count > 0) {
    if (!order || !S || !Y || !sy || !yy) return PMR_E_INVALID;
    unsigned long long seen = 0;
    for (int j = 0; j < count; ++j) {
      if (order[j] < 0 || order[j] >= m || (seen >> order[j]) & 1ull) return PMR_E_INVALID;
      seen |= 1ull << order[j];
    }
  }
  double* w = (double*)work;
  launch_lbfgs_direction(n, m, count, order, S, Y, sy, yy, g, d, w, w + 3 * DOT_BLOCKS + 64,
                         w + vec_work_doubles(n), (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? PMR_OK : PMR_E_HIP;
}

int pmr_lbfgs_direction_noalloc(size_t n, int m, int count, const int* order, const float* S,
                                const float* Y, const double* sy, const double* yy,
                                const float* g, float* d, void* stream) {
  if (!g || !d || n == 0 || g == d || m < 1 || count < 0 || count > m) return PMR_E_INVALID;
  if (m > NOALLOC_MAX_M) return PMR_E_SHAPE;  // the fixed scratch holds 64 scalars
  if (count > 0) {
    if (!order || !S || !Y || !sy || !yy) return PMR_E_INVALID;
    unsigned long long seen = 0;
    for (int j = 0; j < count; ++j) {
      if (order[j] < 0 || order[j] >= m || (seen >> order[j]) & 1ull) return PMR_E_INVALID;
      seen |= 1ull << order[j];
    }
  }
  hipStream_t s = (hipStream_t)stream;
  double* w = nullptr;
  const int st = scratch_of(s, &w);
  if (st != PMR_OK) return st;
  launch_lbfgs_direction(n, m, count, order, S, Y, sy, yy, g, d, w,
                         w + 2 * DOT_BLOCKS + NOALLOC_MAX_M, w + 2 * DOT_BLOCKS, s);
  return hipGetLastError() == hipSuccess ? PMR_OK : PMR_E_HIP;
}

size_t pmr_lbfgs_state_bytes(int max_iter) {
  if (max_iter < 1) return 0;
  return sizeof(pmr_lbfgs_state) + (size_t)(max_iter + 1) * (sizeof(double) + sizeof(long long));
}

int pmr_lbfgs_init(size_t n, const pmr_lbfgs_params* params, void* state, const double* loss,
                   const float* g, float* d, const float* S, const float* Y, const double* sy,
                   const double* yy, void* work, void* stream) {
  if (!params || !state || !loss || !g || !d || !S || !Y || !sy || !yy || !work || n == 0 ||
      g == d)
    return PMR_E_INVALID;
  const pmr_lbfgs_params& p = *params;
  if (p.m < 1 || p.m > PMR_LBFGS_MAX_M || p.max_iter < 1 || p.max_halvings < 0 ||
      !(p.c1 > 0.0 && p.c1 < 1.0) || !(p.curvature_eps >= 0.0) || !(p.rel_tol >= 0.0) ||
      p.stop_below != p.stop_below)
    return PMR_E_INVALID;
  hipStream_t s = (hipStream_t)stream;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return PMR_E_HIP;
  if (s && hipStreamGetDevice(s, &dev) != hipSuccess) return PMR_E_HIP;
  int khz = 0;
  if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0)
    return PMR_E_HIP;
  launch_lbfgs_init(n, p, (pmr_lbfgs_state*)state, loss, g, d, S, Y, sy, yy, (double*)work, khz,
                    s);
  return hipGetLastError() == hipSuccess ? PMR_OK : PMR_E_HIP;
}

int pmr_lbfgs_trial(size_t n, const void* state, const float* x, const float* d, float* xt,
                    void* stream) {
  if (!state || !x || !d || !xt || n == 0 || xt == x || xt == d) return PMR_E_INVALID;
  launch_lbfgs_trial(n, (const pmr_lbfgs_state*)state, x, d, xt, (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? PMR_OK : PMR_E_HIP;
}

int pmr_lbfgs_update(size_t n, int m, void* state, const double* loss, float* x, float* g,
                     const float* xt, const float* gt, float* d, float* S, float* Y, double* sy,
                     double* yy, void* work, void* stream) {
  if (!state || !loss || !x || !g || !xt || !gt || !d || !S || !Y || !sy || !yy || !work ||
      n == 0 || m < 1 || m > PMR_LBFGS_MAX_M || g == d || xt == x || gt == g)
    return PMR_E_INVALID;
  launch_lbfgs_update(n, m, (pmr_lbfgs_state*)state, loss, x, g, xt, gt, d, S, Y, sy, yy,
                      (double*)work, (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? PMR_OK : PMR_E_HIP;
}

size_t pmr_power_work_bytes(int nbins) {
  if (nbins < 1) return 0;
  return power_work_doubles(nbins) * sizeof(double);
}

int pmr_power_bins(int n, double box, const void* a, const void* b, int nbins, double* out,
                   void* work, size_t work_bytes, void* stream) {
  if (!a || !b || !out || !work || !(box > 0)) return PMR_E_INVALID;
  if (n < 2 || n > 1024 || (n & (n - 1)) != 0 || nbins < 1 || nbins > 2 * n) return PMR_E_SHAPE;
  if (work_bytes < pmr_power_work_bytes(nbins)) return PMR_E_WORKSPACE;
  launch_power_bins(n, box, (const float2*)a, (const float2*)b, nbins, out, (double*)work,
                    (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? PMR_OK : PMR_E_HIP;
}

}  // extern "C"
