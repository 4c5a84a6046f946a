// Product of an eliminated block's sparse coupling and dense arrow rows with
// the transposed inverse of its diagonal block.
//
// C = B G^T with B the assembled sub-diagonal block: row (k, s) of B holds the
// stencil of node s (13 points; 5 for the diffusion family) once per response,
// so an element of C is a sum of 13 nv products where the dense product took
// b of them.  Bound by the reads of G through L1 (13 nv columns of 64 rows per
// row of C) and the write of C: one block of 2025 rows with four arrow rows
// takes 31 us, nine of 900 rows 42 us, one of 6075 (three responses) 350 us.
// C begins in each row where its stencil does, so the updates, the solves and
// the selected inversion skip the zeros before it (Band).  Together they took a
// 9-point gradient at 30 x 30, nt = 48 from 52.3 to 38.9 ms, f_obj with all
// variances at 45 x 45, nt = 100 from 172 to 143 ms, and a batch with blocks up
// to 6075 rows from 197 to 137 ms.
#include "couple.hpp"
#include "model.hpp"

#include <algorithm>

namespace dl {

namespace {
constexpr int NT = 256;
constexpr int W = CPW_MAX;  // stencil points of a row and response
constexpr int WP = 16;      // their stride in LDS
constexpr int TR = 32;      // rows of a coupling tile
constexpr int TILE_LDS = 64 * (TR + 1);  // doubles
constexpr int RR = 8;       // arrow rows of a workgroup
constexpr int KC = 128;     // columns of G and of the arrow rows at a time
typedef double v2d __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) double* gptr;
typedef const __attribute__((address_space(1))) v2d* gptr2;

__device__ __forceinline__ double fma_t(double a, double b, double c) {
  return __builtin_fma(a, b, c);
}
__device__ __forceinline__ float fma_t(float a, float b, float c) {
  return __builtin_fmaf(a, b, c);
}

// Rows 32 ti .. of C, columns 64 tj .. for tj = tj0, tj0 + J.groups, ...: the
// rows' coefficients are gathered once for all of them.  Half a wave runs along
// the columns (the rows of G), two to a lane: with 8-byte loads the L1 passed
// half as much.  A half has 4 rows, one at a time, whose 13 loads are in flight
// at once.  The terms of an element are added by increasing column of B, one
// multiply-add each, which is the order and rounding of the matrix instructions'
// chain over the dense row; columns of B from the end of the tile on meet
// zeros of G and are left out, so a tile before the stencil's reach only writes
// zeros.
//
// S: type of the sums.  In FP32 storage with one response it is double, B's
// entries are formed again from the model and C is rounded once: log|Q_p| is
// exact there (one diagonal block's), so what FP32 sums and the rounding of a
// stencil of few distinct values do to log|Q_c|, systematic over all rows, would
// be in f.
template <typename T, typename S>
__device__ __forceinline__ void couple_tiles(const CoupleJob& J, int ti, int tj0, double* lds) {
  const int bp = J.bp, ns = J.ns, nv = J.nv, w = J.w;
  const int lane = threadIdx.x & 31, half = threadIdx.x >> 5;
  T* t = (T*)lds;                                // [64 columns][TR + 1]
  S* val = (S*)(lds + TILE_LDS);                 // [nv][TR][WP]
  int* off = (int*)(lds + TILE_LDS + 3 * TR * WP);  // [nv][TR][WP]: column times bp / 64
  const T* B = (const T*)J.B;
  for (int e = threadIdx.x; e < nv * TR * WP; e += NT) {
    const int r = e % TR, q = (e / TR) % WP, kv = e / (TR * WP);
    const int i = ti * TR + r;
    int k = -1;
    if (i < J.b && q < w) {
      k = J.col[(i % ns) * w + q];
      if (k >= 0) k += kv * ns;
    }
    S v = (S)0;
    if (k >= 0) {
      if constexpr (sizeof(S) > sizeof(T)) {
        const int e0 = J.m->sp_ptr[i] + q;  // the stencil is the whole pattern
        v = J.bc[0] * J.m->sp_C[e0] + J.bc[1] * J.m->sp_G[e0] + J.bc[2] * J.m->sp_G2[e0];
      } else {
        v = B[i + (int64_t)k * J.ldb];
      }
    }
    val[(kv * TR + r) * WP + q] = v;
    off[(kv * TR + r) * WP + q] = k >= 0 ? k * (bp / 64) : 0;
  }
  const int klo = J.band.lo(ti * TR, TR, bp);
  __syncthreads();
  for (int tj = tj0; tj < bp / 64; tj += J.groups) {
    const gptr2 G = (gptr2)((gptr)J.G + tj * 64) + lane;
    const int kend = (tj + 1) * 64, oend = kend * (bp / 64);
#pragma unroll 1
    for (int row = half; row < TR; row += NT / 32) {
      S a0 = (S)0, a1 = (S)0;
      if (klo < kend)
#pragma unroll 1
        for (int kv = 0; kv < nv; ++kv) {
          const int at = (kv * TR + row) * WP;
          v2d g[W];
          S v[W];
#pragma unroll
          for (int q = 0; q < W; ++q) {
            const int o = off[at + q];
            v[q] = o < oend ? val[at + q] : (S)0;
            g[q] = G[(int64_t)(o < oend ? o : oend - bp / 64) * 32];
          }
#pragma unroll
          for (int q = 0; q < W; ++q) {
            a0 = fma_t(v[q], (S)g[q].x, a0);
            a1 = fma_t(v[q], (S)g[q].y, a1);
          }
        }
      t[2 * lane * (TR + 1) + row] = (T)a0;
      t[(2 * lane + 1) * (TR + 1) + row] = (T)a1;
    }
    __syncthreads();
    // the stores run along the rows
    const int r = threadIdx.x % TR, c0 = threadIdx.x / TR;
    T* C = (T*)J.C + ti * TR + r + (int64_t)(tj * 64) * J.ldb;
#pragma unroll
    for (int c = 0; c < 64; c += NT / TR)
      C[(int64_t)(c0 + c) * J.ldb] = t[(c0 + c) * (TR + 1) + r];
    __syncthreads();
  }
}

// Columns 32 tj .. of the product of arrow rows r0 .. r0 + RR - 1 (dense): half a
// wave runs along the columns, the eight halves take every eighth k and are
// summed in their order.  KC columns of G are in flight while the KC before them
// are multiplied (with one buffer less, and 64 columns a unit, four rows at b =
// 2025 took 55 us).  Bound by the unit of the last columns, which reads the last
// 32 rows of G.
template <typename T>
__device__ __forceinline__ void arrow_tile(const CoupleJob& J, int tj, int rc, double* lds) {
  const int64_t bp = J.bp;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r0 = rc * RR, j = lane & 31, kh = 2 * wave + (lane >> 5);
  constexpr int UN = KC / 8, PR = KC * RR / NT;
  typedef const __attribute__((address_space(1))) T* rptr;
  const rptr R = (rptr)J.R + r0 + (threadIdx.x & (RR - 1));
  const gptr G = (gptr)J.G + tj * 32 + j;
  const int kend = (tj / 2 + 1) * 64;  // zeros of G from there on
  double acc[RR];
#pragma unroll
  for (int r = 0; r < RR; ++r) acc[r] = 0.0;
  double ga[UN], gb[UN], xa[PR], xb[PR];
  auto load = [&](double (&g)[UN], double (&x)[PR], int k0) {
#pragma unroll
    for (int u = 0; u < UN; ++u) g[u] = G[min(k0 + 8 * u + kh, kend - 1) * bp];
#pragma unroll
    for (int p = 0; p < PR; ++p) {
      const int k = k0 + (threadIdx.x + p * NT) / RR;
      const double v = (double)R[min(k, kend - 1) * J.ldb];
      x[p] = k < kend ? v : 0.0;
    }
  };
  auto stage = [&](const double (&x)[PR], double* buf) {
#pragma unroll
    for (int p = 0; p < PR; ++p) buf[threadIdx.x + p * NT] = x[p];
    __syncthreads();
  };
  auto mul = [&](const double (&g)[UN], const double* buf) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
#pragma unroll
      for (int r = 0; r < RR; ++r)
        acc[r] = __builtin_fma(buf[(8 * u + kh) * RR + r], g[u], acc[r]);
      if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // few LDS reads in flight
    }
  };
  load(ga, xa, 0);
  for (int k = 0; k < kend; k += 2 * KC) {
    stage(xa, lds);
    load(gb, xb, k + KC);
    mul(ga, lds);
    if (k + KC >= kend) break;
    stage(xb, lds + KC * RR);
    load(ga, xa, k + 2 * KC);
    mul(gb, lds + KC * RR);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RR; ++r) lds[(kh * RR + r) * 32 + j] = acc[r];
  __syncthreads();
  T* out = (T*)J.RC + (int64_t)(tj * 32) * J.ldb;
  {
    const int r = threadIdx.x & (RR - 1), c = threadIdx.x / RR;
    double s = lds[r * 32 + c];
#pragma unroll
    for (int h = 1; h < 8; ++h) s += lds[(h * RR + r) * 32 + c];
    out[r0 + r + (int64_t)c * J.ldb] = (T)s;
  }
  // the padding rows of the arrow block
  const int nrc = (J.a + RR - 1) / RR, np = J.ap - nrc * RR;
  if (rc == nrc - 1)
    for (int e = threadIdx.x; e < np * 32; e += NT)
      out[nrc * RR + e % np + (int64_t)(e / np) * J.ldb] = (T)0;
}

template <typename T>
__device__ __forceinline__ void couple_body(const CoupleJob& J, double* lds) {
  const int nb = J.bp / 64;
  const int arrow = J.R ? 2 * nb * ((J.a + RR - 1) / RR) : 0;
  int u = blockIdx.x;
  if (u < arrow) {  // the longest sums first
    const int nrc = (J.a + RR - 1) / RR;
    arrow_tile<T>(J, 2 * nb - 1 - u / nrc, u % nrc, lds);
    return;
  }
  u -= arrow;
  const int nr = J.bp / TR;
  if (!J.B || u >= nr * J.groups) return;
  if constexpr (sizeof(T) == 4) {
    if (J.bc) {
      couple_tiles<T, double>(J, u / J.groups, u % J.groups, lds);
      return;
    }
  }
  couple_tiles<T, T>(J, u / J.groups, u % J.groups, lds);
}
}  // namespace

template <typename T>
__global__ __launch_bounds__(NT, 4) void k_couple(const CoupleJob* __restrict__ jobs) {
  __shared__ __attribute__((aligned(16))) double lds[TILE_LDS + 3 * TR * WP * 3 / 2];
  couple_body<T>(jobs[blockIdx.y], lds);
}

int finalize_couple(CoupleJob* jobs, int count) {
  // up to eight column tiles a workgroup, as long as the launch keeps four
  // workgroups a compute unit
  int64_t tiles = 0;
  for (int i = 0; i < count; ++i)
    if (jobs[i].B) tiles += (int64_t)(jobs[i].bp / TR) * (jobs[i].bp / 64);
  const int per = (int)std::min<int64_t>(8, std::max<int64_t>(1, tiles / 1024));
  int most = 0;
  for (int i = 0; i < count; ++i) {
    const int nb = jobs[i].bp / 64;
    // a multiple of the XCDs: each then reads its own rows of G
    jobs[i].groups = std::max(1, nb / per);
    if (nb >= 8) jobs[i].groups = (jobs[i].groups + 7) / 8 * 8;
    most = std::max(most, (jobs[i].B ? jobs[i].groups * (jobs[i].bp / TR) : 0) +
                              (jobs[i].R ? 2 * nb * ((jobs[i].a + RR - 1) / RR) : 0));
  }
  return most;
}

hipError_t launch_couple(const CoupleJob* jobs, int count, int max_units, bool f32,
                         hipStream_t s) {
  if (count <= 0 || max_units <= 0) return hipSuccess;
  const dim3 grid(max_units, count);
  if (f32) hipLaunchKernelGGL(k_couple<float>, grid, dim3(NT), 0, s, jobs);
  else hipLaunchKernelGGL(k_couple<double>, grid, dim3(NT), 0, s, jobs);
  return hipGetLastError();
}

}  // namespace dl
