// Memory-bound matrix-vector products of the block forward/backward solves
// (HBM-bound: each job streams one dense block once, coalesced, against up to
// SOLVE_RHS right-hand sides at a time).  One launch serves a batch of
// independent jobs (one per matrix of a batch).
//
// All extents are multiples of 64 and all columns start 16-byte aligned, so
// every lane loads 16 bytes at a time (V = 2 doubles or 4 floats of a column).
// What a right-hand side's result is does not depend on how many others share
// the pass: each is summed in the same fixed order.
//
// On the factor of the 45 x 45, nt = 100 model a solve took 3.55 ms: 16.8 us
// (4.1 TB/s) per pair of 2112 x 2048 blocks plus a 4.1 us launch that summed
// the pieces, and four right-hand sides four times that, since each read the
// whole factor.  Now 2.46 ms
// for one (12.9 us a pair and no second launch) and 3.4 ms for four (17.1), of
// about half the bytes (the zeros before a row's first column are passed over).
#include "solve.hpp"

#include <algorithm>

namespace dl {

namespace {
constexpr int NT = 256;
// Columns of a workgroup of the transposed product.  Eight, with four
// right-hand sides, took 19.9 us where four take 17.6 (too few waves).
constexpr int GEMV_T_COLS = 4;
typedef double v2d __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) double gdouble;
template <typename TA> struct Vec;
template <> struct Vec<double> { typedef v2d type; };
template <> struct Vec<float> { typedef v4f type; };

__device__ __forceinline__ double cload(const double* p) {
  return __hip_atomic_load((const gdouble*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void cstore(double* p, double v) {
  __hip_atomic_store((gdouble*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
}  // namespace

// out = beta*base + alpha*A*x.  Workgroup (i, s) of a job: RB = 64 V rows,
// columns s len ..; its four waves take every fourth column, two batches of
// UN loads in flight in each (UN = 16 cost half the waves: 24.6 us for four
// right-hand sides), and are summed in wave order.  With more than one column slice the sums go to `partial` (device-coherent), and the row block's
// last workgroup to finish adds them in slice order: the slices of a block run
// on all XCDs, and a second launch for the sum cost more than the product of a
// small block.  `cnt` counts the finished workgroups of each row block; the
// last one returns it to zero.  tri: A is lower triangular.
template <int R, typename TA>
__device__ void gemv_n_body(const GemvN& g, double* xs, double* sh, int* s_last) {
  constexpr int V = 16 / (int)sizeof(TA), RB = 64 * V, UN = 8;
  typedef typename Vec<TA>::type vec_t;
  const int rb = blockIdx.x, sl = blockIdx.y;
  if (rb * RB >= g.M) return;
  const int len = gemv_slice_len(g.K);
  const int kend = g.tri ? min(g.K, rb * RB + RB) : g.K;
  // A's zeros before its rows' first column are skipped by whole slices and
  // by whole stages of a slice
  const int klo = min(g.band.lo(rb * RB, min(RB, g.M - rb * RB), g.K), kend - 1);
  const int sl0 = klo / len, nsl = (kend + len - 1) / len - sl0;
  if (sl < sl0 || sl >= sl0 + nsl) return;
  const int k0 = sl * len, k1 = min(kend, k0 + len);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = rb * RB + lane * V;
  const bool ok = row < g.M;
  const TA* p = (const TA*)g.A + (ok ? row : 0) + (int64_t)k0 * g.lda;
  const int n = k1 - k0;
  // tri: columns from the end of the row's 64 x 64 diagonal tile on count as zero
  const int lim = g.tri ? (row | 63) + 1 - k0 : n;
  double acc[R][V];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int v = 0; v < V; ++v) acc[r][v] = 0.0;
  // the slice's x, R values a column, staged GEMV_STAGE columns at a time (slices
  // are 64 columns, or K / GEMV_KS beyond 2048)
  const int kb0 = max(klo - k0, 0) / GEMV_STAGE * GEMV_STAGE;
  for (int kb = kb0; kb < n; kb += GEMV_STAGE) {
    const int nb = min(GEMV_STAGE, n - kb);
    // two batches of columns: the second is in flight while the first is used
    vec_t a[2][UN];
    auto load = [&](vec_t (&d)[UN], int k) {
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int c = gemv_column(k + 4 * u + wave, nb);
        d[u] = *(const __attribute__((address_space(1))) vec_t*)(p + (int64_t)(kb + c) * g.lda);
      }
    };
    auto use = [&](const vec_t (&d)[UN], int k) {
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int c = k + 4 * u + wave;
        if (c < nb) {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const double x = xs[c * R + r];
#pragma unroll
            for (int v = 0; v < V; ++v)
              acc[r][v] = __builtin_fma(kb + c < lim ? (double)d[u][v] : 0.0, x, acc[r][v]);
          }
        }
      }
    };
    load(a[0], 0);
    load(a[1], 4 * UN);
    if (kb > kb0) __syncthreads();
    for (int e = threadIdx.x; e < nb * R; e += NT)
      xs[e] = g.x[k0 + kb + e / R + (int64_t)(e % R) * g.sx];
    __syncthreads();
    for (int k = 0; k < nb; k += 8 * UN) {
      use(a[0], k);
      if (k + 8 * UN < nb) load(a[0], k + 8 * UN);
      use(a[1], k + 4 * UN);
      if (k + 12 * UN < nb) load(a[1], k + 12 * UN);
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int v = 0; v < V; ++v) sh[(wave * R + r) * RB + lane * V + v] = acc[r][v];
  __syncthreads();
  auto wave_sum = [&](int e) {  // e = r RB + row of the block
    return (sh[e] + sh[R * RB + e]) + (sh[2 * R * RB + e] + sh[3 * R * RB + e]);
  };
  if (nsl > 1) {
    for (int e = threadIdx.x; e < R * RB; e += NT) {
      const int m = rb * RB + e % RB;
      if (m < g.M) cstore(&g.partial[((int64_t)sl * R + e / RB) * g.M + m], wave_sum(e));
    }
    __builtin_amdgcn_s_waitcnt(0);  // in every lane, before the count below
    __syncthreads();
    if (threadIdx.x == 0) *s_last = atomicAdd(&g.cnt[rb], 1) == nsl - 1;
    __syncthreads();
    if (!*s_last) return;
    if (threadIdx.x == 0) g.cnt[rb] = 0;
  }
  const int split = g.split < 0 ? g.M : g.split;
  for (int e = threadIdx.x; e < R * RB; e += NT) {
    const int m = rb * RB + e % RB, r = e / RB;
    if (m >= g.M) continue;
    double s;
    if (nsl > 1) {
      s = 0.0;
      for (int q0 = sl0; q0 < sl0 + nsl; q0 += 16) {
        double v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q)
          v[q] = q0 + q < sl0 + nsl ? cload(&g.partial[((int64_t)(q0 + q) * R + r) * g.M + m])
                                    : 0.0;
#pragma unroll
        for (int q = 0; q < 16; ++q) s += v[q];
      }
    } else {
      s = wave_sum(e);
    }
    if (m < split) {
      const double b = g.base1 ? g.beta * g.base1[m + r * g.sb1] : 0.0;
      g.out1[m + r * g.so1] = b + g.alpha * s;
    } else {
      const double b = g.base2 ? g.beta * g.base2[m - split + r * g.s2] : 0.0;
      g.out2[m - split + r * g.s2] = b + g.alpha * s;
    }
  }
}

template <int R>
__global__ __launch_bounds__(NT) void k_gemv_n(const GemvN* __restrict__ jobs) {
  __shared__ double xs[GEMV_STAGE * R];
  __shared__ double sh[4 * R * 256];
  __shared__ int s_last;
  const GemvN g = jobs[blockIdx.z];
  if (g.a32) gemv_n_body<R, float>(g, xs, sh, &s_last);
  else gemv_n_body<R, double>(g, xs, sh, &s_last);
}

hipError_t launch_gemv_n(const GemvN* jobs, int count, int max_M, int max_K, int nrhs,
                         hipStream_t s) {
  if (count <= 0 || max_M <= 0) return hipSuccess;
  // the most slices of any K up to max_K
  const int max_slices = std::min(GEMV_KS, (max_K + 63) / 64);
  const dim3 grid((max_M + 127) / 128, max_slices, count);
  if (nrhs > 1) hipLaunchKernelGGL(k_gemv_n<SOLVE_RHS>, grid, dim3(NT), 0, s, jobs);
  else hipLaunchKernelGGL(k_gemv_n<1>, grid, dim3(NT), 0, s, jobs);
  return hipGetLastError();
}

// y = beta*base + alpha*A^T*x: a workgroup takes TC columns, so that x is
// read once for all of them; its four waves take every fourth RB = 64 V rows
// (lanes along the rows), and each column is summed over the lanes by a fixed
// butterfly and then in wave order.  tri: A is lower triangular.  y must not
// alias x.
template <int R, typename TA>
__device__ void gemv_t_body(const GemvT& g, double* sh) {
  constexpr int V = 16 / (int)sizeof(TA), RB = 64 * V, TC = GEMV_T_COLS;
  typedef typename Vec<TA>::type vec_t;
  const int j0 = blockIdx.x * TC;
  if (j0 >= g.N) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int split = g.split < 0 ? g.M : g.split;
  const TA* A = (const TA*)g.A + (int64_t)j0 * g.lda;
  double acc[R][TC];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < TC; ++c) acc[r][c] = 0.0;
  const int i0 = g.tri ? (j0 / RB) * RB : 0;
  int i = i0 + wave * RB + lane * V;
  if (g.tri && i < (j0 & ~63)) i += 4 * RB;  // above the columns' diagonal tile
#pragma unroll 2
  for (; i < g.M; i += 4 * RB) {
    const int ib = __builtin_amdgcn_readfirstlane(i - lane * V);
    if (g.band.lo(ib, min(RB, g.M - ib), g.N) >= j0 + TC) continue;  // zeros here
    vec_t a[TC];
#pragma unroll
    for (int c = 0; c < TC; ++c)
      a[c] = *(const __attribute__((address_space(1))) vec_t*)(A + i + (int64_t)c * g.lda);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double* x = i < split ? g.x1 + r * g.sx1 + i : g.x2 + r * g.sx2 + (i - split);
      double xv[V];
#pragma unroll
      for (int v = 0; v < V; v += 2) {
        const v2d t = *(const __attribute__((address_space(1))) v2d*)(x + v);
        xv[v] = t.x;
        xv[v + 1] = t.y;
      }
#pragma unroll
      for (int c = 0; c < TC; ++c)
#pragma unroll
        for (int v = 0; v < V; ++v) acc[r][c] = __builtin_fma((double)a[c][v], xv[v], acc[r][c]);
    }
  }
  // a butterfly over the lanes, halving the sums a lane carries while it has
  // several: R TC - 1 + 6 - log2(R TC) exchanges in place of 6 R TC
  double* a = &acc[0][0];
  int held = 0;  // the sum this lane ends up with
#pragma unroll
  for (int off = 32, n = R * TC; off > 0; off >>= 1) {
    const bool up = lane & off;
    if (n > 1) {
      n >>= 1;
#pragma unroll
      for (int e = 0; e < n; ++e) {
        const double keep = up ? a[e + n] : a[e];
        a[e] = keep + __shfl_xor(up ? a[e] : a[e + n], off, 64);
      }
      held += up ? n : 0;
    } else {
      a[0] += __shfl_xor(a[0], off, 64);
    }
  }
  // every sum once: the lanes below its last exchange hold copies
  if ((lane & (64 / (R * TC) - 1)) == 0) sh[wave * R * TC + held] = a[0];
  __syncthreads();
  if (threadIdx.x < R * TC) {
    const int r = threadIdx.x / TC, j = j0 + threadIdx.x % TC;
    constexpr int E = R * TC;
    const int e = threadIdx.x;
    const double s = (sh[e] + sh[E + e]) + (sh[2 * E + e] + sh[3 * E + e]);
    const double b = g.base ? g.beta * g.base[j + r * g.sb] : 0.0;
    g.y[j + r * g.sy] = b + g.alpha * s;
  }
}

template <int R>
__global__ __launch_bounds__(NT) void k_gemv_t(const GemvT* __restrict__ jobs) {
  __shared__ double sh[4 * R * GEMV_T_COLS];
  const GemvT g = jobs[blockIdx.y];
  if (g.a32) gemv_t_body<R, float>(g, sh);
  else gemv_t_body<R, double>(g, sh);
}

hipError_t launch_gemv_t(const GemvT* jobs, int count, int max_N, int nrhs, hipStream_t s) {
  if (count <= 0 || max_N <= 0) return hipSuccess;
  const dim3 grid((max_N + GEMV_T_COLS - 1) / GEMV_T_COLS, count);
  if (nrhs > 1) hipLaunchKernelGGL(k_gemv_t<SOLVE_RHS>, grid, dim3(NT), 0, s, jobs);
  else hipLaunchKernelGGL(k_gemv_t<1>, grid, dim3(NT), 0, s, jobs);
  return hipGetLastError();
}

}  // namespace dl
