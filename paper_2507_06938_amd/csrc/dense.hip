// Small dense kernels: 64x64 diagonal-tile Cholesky + inverse, tile copies,
// fills, deterministic log-sum reductions.
#include "common.hpp"

#define DL_DAG_FN __host__ __device__ inline
#include "dag.hpp"

namespace dl {

namespace {
constexpr int NB = 64;
constexpr int LDL = NB + 2;         // LDS row stride: 528 B, 16-byte aligned rows
constexpr int TILE_LDS = NB * LDL;  // doubles of one staged 64 x 64 tile
constexpr int POTRF_NT = 1024;      // threads of a tile-factor workgroup (16 waves)
typedef double v4d __attribute__((ext_vector_type(4)));
}

// Device-coherent accesses (agent-scope relaxed atomics: sc1 loads and
// stores that bypass the per-XCD caches): the persistent factorisation
// exchanges tiles between workgroups on different XCDs with these.
// (global address space: keeps them off the generic load path)
typedef __attribute__((address_space(1))) double gdouble;
__device__ __forceinline__ double cload(const double* p) {
  return __hip_atomic_load((const gdouble*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void cstore(double* p, double v) {
  __hip_atomic_store((gdouble*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// p must point to global memory
__device__ __forceinline__ double global_load(const double* p) { return *(const gdouble*)p; }
__device__ __forceinline__ void global_store(double* p, double v) { *(gdouble*)p = v; }
template <bool COH>
__device__ __forceinline__ void gstore(double* p, double v) {
  if constexpr (COH) cstore(p, v);
  else *p = v;
}

// 1/sqrt(x) for x > 0: hardware estimate (relative error e0 below 2^-20)
// refined by one cubic step y (1 + e/2 + 3/8 e^2), e = 1 - x y^2, which leaves
// 5/16 e^3 = 5/2 e0^3 before rounding: four dependent operations where two
// Newton steps take six.
__device__ __forceinline__ double rsqrt_nr(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = __builtin_fma(-(x * y), y, 1.0);
  return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}

// One 16x16 block of a product of LDS tiles stored S[k*LDL + c]:
//   D[a][b] = sum_{k < kmax} P[k][p0 + a] Q[k][q0 + b],
// on v_mfma_f64_16x16x4_f64 (lane l supplies P[k0 + l/16][p0 + l%16] as the
// "A" operand and Q[k0 + l/16][q0 + l%16] as "B"; register r of lane l
// receives D[l/16 + 4r][l%16]).  kmax: multiple of 4, at most 64.
__device__ __forceinline__ void mfma1_k64(const double* P, int p0, const double* Q,
                                          int q0, v4d& acc, int kmax = NB) {
  const int l = threadIdx.x & 63;
  const int lr = l & 15, lk = l >> 4;
#pragma unroll 4
  for (int k0 = 0; k0 < kmax; k0 += 4) {
    const double a = P[(k0 + lk) * LDL + p0 + lr];
    const double b = Q[(k0 + lk) * LDL + q0 + lr];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
  }
}

// threadIdx.x and this lane's index in its wave as values of their own at each
// place: address arithmetic on them is then not kept in registers over the
// long bodies around it (the tile kernels have 128 registers a lane)
__device__ __forceinline__ int thread_index() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
__device__ __forceinline__ int lane_index() { return thread_index() & 63; }

// ---- one 16-column panel of the tile factor, by one wave --------------------------------
//
// Lane i holds row i % 16 of the panel's 16 x 16 diagonal block in rd (every
// group of 16 lanes has all of it) and one row of the panel's other rows in
// rp: X L^T = B row by row.  The factor L(c, q) that the update of column c
// needs is in lane c of each group's rd[q], and the FP64 FMA takes it from
// there itself (DPP row_newbcast: lane N of a row of 16 to the whole row), one
// instruction per update.  Reading it into a scalar (v_readlane, two per
// factor) stalls the wave for about 16 cycles per use.  A VALU result must be
// two wait states old when a DPP operand reads it; the statements are volatile
// and so stay in order, and the ones that can come right after their operand's
// definition carry the wait.
template <int LANE>
__device__ __forceinline__ double row_bcast(double x) {
  double r;
  asm volatile("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf"
               : "=v"(r)
               : "v"(x), "n"(LANE));
  return r;
}

// rd[C] -= L(C, Q) rd[Q] and rp[C] -= L(C, Q) rp[Q]
template <int Q, int C>
__device__ __forceinline__ void panel_update(double (&rd)[16], double (&rp)[16]) {
  if constexpr (C == Q + 1)
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f64_dpp %0, %2, -%2 row_newbcast:%4 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %1, %2, -%3 row_newbcast:%4 row_mask:0xf bank_mask:0xf"
                 : "+v"(rd[C]), "+v"(rp[C])
                 : "v"(rd[Q]), "v"(rp[Q]), "n"(C));
  else
    asm volatile("v_fmac_f64_dpp %0, %2, -%2 row_newbcast:%4 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %1, %2, -%3 row_newbcast:%4 row_mask:0xf bank_mask:0xf"
                 : "+v"(rd[C]), "+v"(rp[C])
                 : "v"(rd[Q]), "v"(rp[Q]), "n"(C));
}
template <int Q, int C>
__device__ __forceinline__ void panel_updates(double (&rd)[16], double (&rp)[16]) {
  if constexpr (C < 16) {
    panel_update<Q, C>(rd, rp);
    panel_updates<Q, C + 1>(rd, rp);
  }
}

// Columns Q .. 15 of the panel, d the pivot of column Q.  A pivot that is not
// positive makes its whole column NaN, and all later ones.  Column Q + 1 is
// updated first, so that its pivot's chain overlaps the updates of the columns
// after it.
template <int Q>
__device__ __forceinline__ void panel_columns(double (&rd)[16], double (&rp)[16], double d) {
  const double rs = rsqrt_nr(d);
  rd[Q] *= rs;
  rp[Q] *= rs;
  if constexpr (Q + 1 < 16) {
    panel_update<Q, Q + 1>(rd, rp);
    d = row_bcast<Q + 1>(rd[Q + 1]);
    panel_updates<Q, Q + 2>(rd, rp);
    panel_columns<Q + 1>(rd, rp, d);
  }
}

// Cholesky A = L L^T of one 64 x 64 SPD tile and G = L^{-1}, by one
// workgroup of 16 waves, in four panels of 16 columns.  What bounds it is the
// chain of 64 pivots (each: broadcast, reciprocal square root, scaling, update
// of the next column), so one wave runs a whole panel in its registers with
// no barrier inside it, and everything that is a product runs on the matrix
// cores of the other waves, where it hides behind the next panel:
//  * panel p, wave 0 (panel_columns): the diagonal block, the rows below it and,
//    as 16 more right-hand rows (those of the identity, solved to L_pp^-T), the
//    block's inverse;
//  * after it, one 16 x 16 block per wave: the trailing blocks A_IJ -= L_Ip
//    L_Jp^T, and row p of the inverse, G_pj = -G_pp T_pj (j < p);
//  * beside panel p + 1: T_rj += L_rp G_pj for the rows r > p below, and (p =
//    2) the first 48 rows of G are stored.
// A panel takes about 2 300 cycles (145 a pivot), by the issue of its 240
// multiply-adds with a broadcast operand: the reciprocal root's steps laid between
// them changed nothing, a broadcast move before two plain multiply-adds took 744 us
// for 711 (32 tiles of the dense entry).  One 4-column panel per wave
// and 16 hand-overs through LDS took 420 cycles a pivot: the launch of one tile
// went from 12.7 to 10.0 us, a panel step's launch from 21.6 to 18.0 us, a
// persistent launch over two blocks of 32 tiles from 783 to 693 us.
//
// src/lds: the tile (column-major, global), copied to Lc first; null when the
// caller has it in Lc already (Lc[k*LDL + i] = A(i, k), after a barrier).
// Lc, Gk: two LDS tiles of TILE_LDS doubles; on return (after a barrier) Lc
// holds L as it held A and Gk[k*LDL + c] = G(k, c), both in the lower triangle
// (other entries are undefined).  Outputs as described for PotrfTileArgs (A/lda: where mode 0
// writes L and mode 1 writes G).
// COH: G (and L) are stored device-coherent.
template <bool COH = false>
__device__ __forceinline__ void potrf_body(const double* src, int64_t lds, double* Lc,
                                           double* Gk, double* A, int64_t lda,
                                           double* Ginv, double* logdiag, int64_t* info,
                                           int64_t row0, int mode) {
  constexpr int PW = 16, NP = NB / PW;  // panel width, panels
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double* const dst = mode == 0 ? Ginv : A;
  const int64_t ldd = mode == 0 ? NB : lda;
  if (src) {
#pragma unroll
    for (int e = 0; e < NB * NB / POTRF_NT; ++e) {
      const int idx = threadIdx.x + e * POTRF_NT;
      Lc[(idx >> 6) * LDL + (idx & 63)] = src[(idx & 63) + (idx >> 6) * lds];
    }
    __syncthreads();
  }
  // 16 x 16 block (block row, block column) of a product of LDS operands
  // stored k-major: acc[a][b] += sum_k P(k, a) Q(k, b) over 16 k
  auto mm = [](const double* P, int ps, const double* Q, int qs, int lk, v4d acc) {
#pragma unroll
    for (int k0 = 0; k0 < PW; k0 += 4)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(P[(k0 + lk) * ps], Q[(k0 + lk) * qs], acc, 0,
                                                 0, 0);
    return acc;
  };
#pragma unroll 1
  for (int p = 0; p < NP; ++p) {
    const int c0 = PW * p;
    const int i = lane_index();
    const int lr = i & 15, lk = i >> 4;
    if (wv == 0) {
      // lane group g: the identity (g = 0), rows 16 (p + g) .. below the
      // diagonal block, or rows above it (whose results nobody reads)
      const int row = PW * ((p + lk) & (NP - 1)) + lr;
      double rd[PW], rp[PW];
#pragma unroll
      for (int q = 0; q < PW; ++q) rd[q] = Lc[(c0 + q) * LDL + c0 + lr];
#pragma unroll
      for (int q = 0; q < PW; ++q) rp[q] = Lc[(c0 + q) * LDL + row];
      if (lk == 0) {
#pragma unroll
        for (int q = 0; q < PW; ++q) rp[q] = lr == q ? 1.0 : 0.0;
      }
      panel_columns<0>(rd, rp, row_bcast<0>(rd[0]));
      double* const out = (lk == 0 ? Gk : Lc) + c0 * LDL + row;
#pragma unroll
      for (int q = 0; q < PW; ++q) out[q * LDL] = rp[q];
      if (lk == 0) {
#pragma unroll
        for (int q = 0; q < PW; ++q) Lc[(c0 + q) * LDL + row] = rd[q];
      }
    } else if (p > 0) {
      // T_rj += L_r,p-1 G_p-1,j, r >= p, j < p (three or four blocks, on waves
      // that share no SIMD with wave 0)
      const int t = wv < 4 ? wv - 1 : (wv == 5 ? 3 : NB);
      if (t < (NP - p) * p) {
        const int up = p == 1 ? t : (p == 2 ? t >> 1 : 0);  // t / p
        const int rb = PW * (p + up), jb = PW * (t - up * p), kb = c0 - PW;
        double* T = Gk + rb * LDL + jb;
        v4d acc = {0.0, 0.0, 0.0, 0.0};
        if (jb < kb) {
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] = T[(lk + 4 * e) * LDL + lr];
        }
        acc = mm(Lc + kb * LDL + rb + lr, LDL, Gk + kb * LDL + jb + lr, LDL, lk, acc);
#pragma unroll
        for (int e = 0; e < 4; ++e) T[(lk + 4 * e) * LDL + lr] = acc[e];
      } else if (p == NP - 1 && wv >= 4 && dst) {
        // the rows of G above the last panel's, by 12 waves
        constexpr int R0 = NB - PW;
        for (int idx = threadIdx.x - 256; idx < R0 * NB; idx += POTRF_NT - 256) {
          const int rr = idx % R0, cc = idx / R0;
          gstore<COH>(&dst[rr + cc * ldd], (rr >= cc) ? Gk[rr * LDL + cc] : 0.0);
        }
      }
    }
    __syncthreads();
    const int nt = NP - 1 - p, nu = nt * (nt + 1) / 2;
    if (wv < nu) {
      // trailing block (I, J), the next panel's column first
      int J = 0, u = wv;
      while (u >= nt - J) {
        u -= nt - J;
        ++J;
      }
      const int ib = PW * (p + 1 + J + u), jb = PW * (p + 1 + J);
      double* C = Lc + jb * LDL + ib;
      v4d old, acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int e = 0; e < 4; ++e) old[e] = C[(lk + 4 * e) * LDL + lr];
      acc = mm(Lc + c0 * LDL + jb + lr, LDL, Lc + c0 * LDL + ib + lr, LDL, lk, acc);
#pragma unroll
      for (int e = 0; e < 4; ++e) C[(lk + 4 * e) * LDL + lr] = old[e] - acc[e];
    } else if (wv < nu + p) {
      const int jb = PW * (wv - nu);
      double* T = Gk + c0 * LDL + jb;
      v4d acc = {0.0, 0.0, 0.0, 0.0};
      acc = mm(Gk + (c0 + lr) * LDL + c0, 1, T + lr, LDL, lk, acc);
#pragma unroll
      for (int e = 0; e < 4; ++e) T[(lk + 4 * e) * LDL + lr] = -acc[e];
    }
    __syncthreads();
  }
  const int i = lane_index();
  if (wv == 15) {
    // the first column that is not a number is the first bad pivot
    const double d = Lc[i * LDL + i];
    if (logdiag) logdiag[i] = log(d);
    const unsigned long long nan = __ballot(!(d > 0.0));
    if (nan && info && i == 0)
      atomicCAS((unsigned long long*)info, 0ull, (unsigned long long)(row0 + __ffsll(nan)));
  }
  if (mode == 0) {
    for (int idx = threadIdx.x; idx < NB * NB; idx += POTRF_NT) {
      const int rr = idx & 63, cc = idx >> 6;
      A[rr + (int64_t)cc * lda] = (rr >= cc) ? Lc[cc * LDL + rr] : 0.0;
    }
  }
  if (dst) {
    constexpr int R0 = NB - PW;
    const int rr = R0 + (threadIdx.x & 15), cc = threadIdx.x >> 4;
    gstore<COH>(&dst[rr + cc * ldd], (rr >= cc) ? Gk[rr * LDL + cc] : 0.0);
  }
}

__global__ __launch_bounds__(POTRF_NT) void k_potrf_tile(const PotrfTileArgs* __restrict__ args) {
  const PotrfTileArgs a = args[blockIdx.x];
  __shared__ __align__(16) double Lc[TILE_LDS];
  __shared__ __align__(16) double Gk[TILE_LDS];
  potrf_body(a.A, a.lda, Lc, Gk, a.A, a.lda, a.Ginv, a.logdiag, a.info, a.row0, a.mode);
}

hipError_t launch_potrf_tiles(const PotrfTileArgs* args, int count,
                              hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_potrf_tile, dim3(count), dim3(POTRF_NT), 0, s, args);
  return hipGetLastError();
}

constexpr int DPER = NB * NB / POTRF_NT;  // elements of a tile per lane

// The lane's DPER elements of the 64 x 64 tile X (global, ld): element idx =
// threadIdx.x + e * POTRF_NT is X(idx & 63, idx >> 6).  All loads are issued
// before any is used.
template <bool COH>
__device__ __forceinline__ void tile_regs(const double* __restrict__ X, int64_t ld,
                                          double (&v)[DPER]) {
  const int tid = thread_index();
#pragma unroll
  for (int e = 0; e < DPER; ++e) {
    const int idx = tid + e * POTRF_NT;
    const double* p = &X[(idx & 63) + (int64_t)(idx >> 6) * ld];
    v[e] = COH ? cload(p) : global_load(p);
  }
}
// S[k*LDL + r] = X(r, k)
__device__ __forceinline__ void regs_to_cols(const double (&v)[DPER], double* S) {
  const int tid = thread_index();
#pragma unroll
  for (int e = 0; e < DPER; ++e) {
    const int idx = tid + e * POTRF_NT;
    S[(idx >> 6) * LDL + (idx & 63)] = v[e];
  }
}
// S[k*LDL + r] = X(k, r) (the transpose)
__device__ __forceinline__ void regs_to_rows(const double (&v)[DPER], double* S) {
  const int tid = thread_index();
#pragma unroll
  for (int e = 0; e < DPER; ++e) {
    const int idx = tid + e * POTRF_NT;
    S[(idx & 63) * LDL + (idx >> 6)] = v[e];
  }
}

// ---- fused panel step ---------------------------------------------------------------
//
// Per tile, with the 64 x 64 operands staged in LDS (S0 = L(I, j), S2 =
// L(J, j)):  A(I, J) -= L(I, j) L(J, j)^T  on FP64 MFMA, one 16 x 16 block
// per wave, with the operand roles chosen so that a lane's results lie along
// the rows of the column-major output (coalesced stores).  Every global load
// (the operand tiles and the elements a lane updates) is issued before the
// first LDS store, so their latencies overlap.  The factoring workgroup
// stages its updated tile in LDS (S1) and runs the tile factor on it with S0
// and S2 as scratch.  A column workgroup also updates the diagonal tile j+1
// (from L(J, j) in S2: the factoring workgroup's product, bit for bit),
// factors it in LDS without writing it, and stores L(I, j+1) = A(I, j+1) G^T
// in place of its tile.  The inverse's workgroups form one or two tile
// products each (see PanelTask).

__device__ __forceinline__ double* stage_tile(const PanelTask& T, int r, int c) {
  return T.stage + ((int64_t)(r * (r - 1) / 2 + c)) * (NB * NB);
}

// The inverse's workgroups of step j (role 2: row j, column c; role 3:
// accumulator (r, c), r > j).  With X(r', c) the product Y X^T of staged
// tiles (mfma1_k64), lane results lie at (q0 + lr, p0 + lk + 4 rg).
__device__ void panel_inverse(const PanelTask& T, int role, int loc, double* S0, double* S1) {
  const int j = T.j;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = lane_index();
  const int lr = l & 15, lk = l >> 4;
  const int p0 = 16 * (wv >> 2), q0 = 16 * (wv & 3);
  const int64_t ld = T.ld;
  double* const A = T.A;
  auto tileA = [&](int r, int c) { return A + (int64_t)r * NB + (int64_t)c * NB * ld; };
  const int r = (role == 2) ? j : j + 1 + loc / j;
  const int c = (role == 2) ? loc : loc % j;
  // G(j-1, c): the diagonal tile, the staged G(j-1, j-2), or in place
  const double* Gk;
  int64_t ldg;
  if (c == j - 1) { Gk = tileA(j - 1, j - 1); ldg = ld; }
  else if (c == j - 2) { Gk = stage_tile(T, j - 1, j - 2); ldg = NB; }
  else { Gk = tileA(j - 1, c); ldg = ld; }
  double prev[4] = {0.0, 0.0, 0.0, 0.0};
  if (c <= j - 2) {
    const double* Sp = stage_tile(T, r, c);
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) prev[rg] = global_load(&Sp[(q0 + lr) + (p0 + lk + 4 * rg) * NB]);
  }
  double vy[DPER], vx[DPER], vg[DPER];
  tile_regs<false>(tileA(r, j - 1), ld, vy);  // Y = L(r, j-1)
  tile_regs<false>(Gk, ldg, vx);              // X = G(j-1, c)^T
  // G_jj, for the second product: from the side ring during the panel steps,
  // in place for the closing launch
  if (role == 2) tile_regs<false>(T.last ? tileA(j, j) : T.gside + (int64_t)(j & 1) * NB * NB,
                                  T.last ? ld : NB, vg);
  if (role == 2 && c == 0 && j >= 2) {
    // G(j-1, j-2) from stage into place (L(j-1, j-2) is read no more)
    const double* src = stage_tile(T, j - 1, j - 2);
    double* dst = tileA(j - 1, j - 2);
    for (int idx = threadIdx.x; idx < NB * NB; idx += POTRF_NT)
      global_store(&dst[(idx & 63) + (int64_t)(idx >> 6) * ld], global_load(&src[idx]));
  }
  regs_to_cols(vy, S0);
  regs_to_rows(vx, S1);
  __syncthreads();
  v4d t = {prev[0], prev[1], prev[2], prev[3]};
  mfma1_k64(S1, p0, S0, q0, t);         // t = S(r, c) + L(r, j-1) G(j-1, c)
  if (role == 3) {
    double* Sd = stage_tile(T, r, c);
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) global_store(&Sd[(q0 + lr) + (p0 + lk + 4 * rg) * NB], t[rg]);
    return;
  }
  // G(j, c) = -G_jj t
  __syncthreads();  // S0, S1 are read no more
  regs_to_cols(vg, S0);                 // Y = G_jj
#pragma unroll
  for (int rg = 0; rg < 4; ++rg) S1[(q0 + lr) * LDL + p0 + lk + 4 * rg] = t[rg];  // X = t^T
  __syncthreads();
  v4d g = {0.0, 0.0, 0.0, 0.0};
  mfma1_k64(S1, p0, S0, q0, g, q0 + 16);  // G_jj is lower triangular
  double* dst;
  int64_t ldd;
  if (c == j - 1) { dst = stage_tile(T, j, j - 1); ldd = NB; }
  else { dst = tileA(j, c); ldd = ld; }
#pragma unroll
  for (int rg = 0; rg < 4; ++rg)
    global_store(&dst[(q0 + lr) + (int64_t)(p0 + lk + 4 * rg) * ldd], -g[rg]);
}

__global__ __launch_bounds__(POTRF_NT) void k_panel_update(const PanelTask* __restrict__ step) {
  __shared__ __align__(16) double pool[3 * TILE_LDS];
  double* S0 = pool;
  double* S1 = pool + TILE_LDS;
  double* S2 = pool + 2 * TILE_LDS;
  // role segments: 0 factor, 1 column, 2 inverse row, 3 inverse accumulate, 4 rest
  int loc = blockIdx.x, role = 0;
  while (role < 4 && loc >= step->tot[role]) {
    loc -= step->tot[role];
    ++role;
  }
  const PanelTask T = *step;
  if (role == 2 || role == 3) {
    panel_inverse(T, role, loc, S0, S1);
    return;
  }
  int I, J;
  if (role == 0) {
    I = J = 0;
  } else if (role == 1) {
    I = 1 + loc;
    J = 0;
  } else {
    // row-major enumeration of the lower triangle of tiles (I, J), J >= 1
    int R = (int)((sqrt(8.0 * (double)loc + 1.0) - 1.0) * 0.5);
    while ((R + 1) * (R + 2) / 2 <= loc) ++R;
    while (R * (R + 1) / 2 > loc) --R;
    I = R + 1;
    J = loc - R * (R + 1) / 2 + 1;
  }
  const int64_t ti0 = (int64_t)(T.j + 1 + I) * NB, tj0 = (int64_t)(T.j + 1 + J) * NB;
  const int64_t pc = (int64_t)T.j * NB * T.ld;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = lane_index();
  const int lr = l & 15, lk = l >> 4;
  const int p0 = 16 * (wv >> 2), q0 = 16 * (wv & 3);  // this wave's 16 x 16 block
  double* C = T.A + ti0 + tj0 * T.ld;
  const bool diag = (I == J);
  const int64_t co = (q0 + lr) + (int64_t)(p0 + lk) * T.ld;  // element rg at co + 4 rg ld
  double vp[DPER], vq[DPER], cpre[4], dpre[4];
  // every load is issued before the first is used: a tile on the diagonal
  // reads its one operand twice rather than branch, and the factoring and
  // column workgroups load the diagonal tile j+1 into registers of their own
  // (left undefined elsewhere).  With loads through generic pointers and a
  // branch that kept them apart the widest launches took 1.5 times as long
  tile_regs<false>(T.A + ti0 + pc, T.ld, vp);
  tile_regs<false>(T.A + tj0 + pc, T.ld, vq);
#pragma unroll
  for (int rg = 0; rg < 4; ++rg) cpre[rg] = global_load(&C[co + (int64_t)(4 * rg) * T.ld]);
  if (role <= 1) {
    const double* Dj = T.A + (int64_t)(T.j + 1) * NB * (T.ld + 1);
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) dpre[rg] = global_load(&Dj[co + (int64_t)(4 * rg) * T.ld]);
  }
  if (role == 0 && T.j >= 1) {
    // G_j from the side ring into diagonal tile j (read by nobody now)
    const double* src = T.gside + (int64_t)(T.j & 1) * NB * NB;
    double* dst = T.A + (int64_t)T.j * NB * (T.ld + 1);
    for (int idx = threadIdx.x; idx < NB * NB; idx += POTRF_NT)
      global_store(&dst[(idx & 63) + (int64_t)(idx >> 6) * T.ld], global_load(&src[idx]));
  }
  regs_to_cols(vp, S0);
  if (!diag) regs_to_cols(vq, S2);
  __syncthreads();
  // (L_I L_J^T)^T = L_J L_I^T: D[n][m] = sum_c L_J(n, c) L_I(m, c)
  const double* LJ = diag ? S0 : S2;
  v4d u0 = {0.0, 0.0, 0.0, 0.0};
  mfma1_k64(LJ, p0, S0, q0, u0);  // u: update(m = q0 + lr, n = p0 + lk + 4r)
  if (role == 4) {
#pragma unroll
    for (int rg = 0; rg < 4; ++rg)
      global_store(&C[co + (int64_t)(4 * rg) * T.ld], cpre[rg] - u0[rg]);
    return;
  }
  // the diagonal tile j+1, updated by the column workgroups exactly as by the
  // factoring one, and its factor.  While column j+1 below reads diagonal tile
  // j+1, G_{j+1} goes to the ring
  const bool side = T.j + 2 < T.nbk;
  double* dst = side ? T.gside + (int64_t)((T.j + 1) & 1) * NB * NB : C;
  v4d v0 = u0;
  if (role == 1) {
    v0 = (v4d){0.0, 0.0, 0.0, 0.0};
    mfma1_k64(S2, p0, S2, q0, v0);
  }
  __syncthreads();  // S0, S2 are read no more
#pragma unroll
  for (int rg = 0; rg < 4; ++rg)
    S1[(p0 + lk + 4 * rg) * LDL + q0 + lr] = dpre[rg] - v0[rg];
  __syncthreads();
  const bool own = role == 0;
  potrf_body(nullptr, 0, S1, S2, own ? dst : nullptr, side ? NB : T.ld, nullptr,
             own ? T.logdiag : nullptr, own ? T.info : nullptr, T.row0, own && T.inv == PANEL_L ? 0 : 1);
  if (own) return;
  // G staged as S1[k][r] = G(r, k) (zero above the diagonal); the updated
  // panel tile as S0[c][m] = A(m, c)
  for (int idx = threadIdx.x; idx < NB * NB; idx += POTRF_NT) {
    const int r = idx & 63, k = idx >> 6;
    S1[k * LDL + r] = (r >= k) ? S2[r * LDL + k] : 0.0;
  }
#pragma unroll
  for (int rg = 0; rg < 4; ++rg) S0[(p0 + lk + 4 * rg) * LDL + q0 + lr] = cpre[rg] - u0[rg];
  __syncthreads();
  // L^T = G A^T: D[c][m] = sum_k G(c, k) A(m, k), k <= c < p0 + 16
  v4d a0 = {0.0, 0.0, 0.0, 0.0};
  mfma1_k64(S1, p0, S0, q0, a0, p0 + 16);  // L(m = q0 + lr, c = p0 + lk + 4r)
#pragma unroll
  for (int rg = 0; rg < 4; ++rg) global_store(&C[co + (int64_t)(4 * rg) * T.ld], a0[rg]);
}

// Fill the workgroups of each role; return the grid size.
static int panel_grid(PanelTask& t) {
  const int j = t.j, nbk = t.nbk, m = nbk - j - 1;  // m: trailing tile rows
  const bool inv = t.inv == PANEL_INVERSE;
  const int steps[5] = {1, m - 1, inv ? j : 0, inv ? m * j : 0, m * (m - 1) / 2};
  const int last[5] = {0, 0, j, 0, 0};
  int grid = 0;
  for (int k = 0; k < 5; ++k) {
    t.tot[k] = t.last ? last[k] : steps[k];
    grid += t.tot[k];
  }
  return grid;
}

int panel_steps(int64_t n, double* A, int64_t lda, int inv, double* logdiag, int64_t* info,
                double* tmp, PanelTask* t, int* grid) {
  const int nbk = (int)(n / NB), steps = inv == PANEL_INVERSE ? nbk : nbk - 1;
  for (int j = 0; j < steps; ++j) {
    PanelTask& p = t[j];
    p = PanelTask{};
    p.A = A;
    p.ld = lda;
    p.logdiag = logdiag + (int64_t)(j + 1) * NB;
    p.info = info;
    p.row0 = (int64_t)(j + 1) * NB;
    p.gside = tmp;
    p.stage = tmp + 2 * NB * NB;
    p.j = j;
    p.nbk = nbk;
    p.last = j + 1 == nbk;
    p.inv = inv;
    grid[j] = panel_grid(p);
  }
  return steps;
}

hipError_t launch_panel_step(const PanelTask* step, int grid, hipStream_t s) {
  if (grid <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_panel_update, dim3(grid), dim3(POTRF_NT), 0, s, step);
  return hipGetLastError();
}

// ---- persistent tile-task factorisation of diagonal blocks ----------------------------
//
// Workgroups of 16 waves take task words from the launch's list in order
// (one atomic add on head[0] each), wait until the counters the task depends
// on are set (a lane polls each, 2 s limit), run the task on 64 x 64 tiles
// staged in LDS and set the task's counter.  The tile operations
// are those of the panel launches of dl_dpotrf: the same staging, the same
// MFMA products (mfma1_k64), the same tile factor (potrf_body).
//
// Hand-over between workgroups, which may sit on different XCDs (each with
// its own L2), without cache write-back or invalidation: every value a task
// writes for another task (A, G, L and accumulator tiles) is stored
// device-coherently (sc1), and every value that another task may have
// rewritten during the launch (A, G and accumulator tiles) is loaded
// device-coherently.  L tiles are written once per launch, after which
// nobody writes them, and nobody reads them before, so they are read through
// the caches (each is read by many update tasks).  A task's stores are
// complete (s_waitcnt) in every lane before the barrier after which its
// counter is set; the counters themselves are relaxed device-scope atomics.

namespace {
// of the 100 MHz constant clock: 2 s of polling, of which one poll counts 0.1 ms at
// most (it takes about a microsecond)
constexpr long long kDagWaitTicks = 200000000;
constexpr long long kDagPollTicks = 10000;

typedef __attribute__((address_space(1))) int32_t gint;
__device__ __forceinline__ int dag_load(const int32_t* p) {
  return __hip_atomic_load((const gint*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void dag_store(int32_t* p, int v) {
  __hip_atomic_store((gint*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// true once *p >= value; false after kDagWaitTicks of polling, or at once when the
// launch has given up (*abort set by a wait that timed out)
__device__ bool dag_wait(const int32_t* p, int value, int32_t* abort) {
  if (dag_load(p) >= value) return true;
  dag::Patience patience{wall_clock64()};
  for (;;) {
    __builtin_amdgcn_s_sleep(1);
    if (dag_load(p) >= value) return true;
    if (dag_load(abort) != 0) return false;
    if (patience.out(wall_clock64(), kDagWaitTicks, kDagPollTicks)) {
      dag_store(abort, 1);
      return false;
    }
  }
}

}  // namespace

__global__ __launch_bounds__(POTRF_NT) void k_dag_chol(const DagTask* __restrict__ tasks,
                                                       int ntask,
                                                       const DagBlock* __restrict__ blocks,
                                                       int nblocks, int32_t* head) {
  __shared__ __align__(16) double pool[4 * TILE_LDS];
  __shared__ int s_task, s_last;
  double* S0 = pool;
  double* S1 = pool + TILE_LDS;
  double* S2 = pool + 2 * TILE_LDS;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int p0 = 16 * (wv >> 2), q0 = 16 * (wv & 3);  // this wave's 16 x 16 block
  if (threadIdx.x == 0) s_task = atomicAdd(head, 1);
  __syncthreads();
  for (;;) {
    const int l = lane_index();
    const int lr = l & 15, lk = l >> 4;
    const int ti = __builtin_amdgcn_readfirstlane(s_task);
    if (ti >= ntask) break;
    int bi = 0;
    const DagTask* rec = tasks + ti;
    const dag::Task t = dag::unpack(rec->word, &bi);
    const DagBlock B = blocks[bi];
    const int64_t ld = B.ld;
    auto tile = [&](double* base, int r, int c) {
      return base + (int64_t)r * NB + (int64_t)c * NB * ld;
    };
    auto tileL = [&](int r, int c) {
      return B.L + ((int64_t)r * (r - 1) / 2 + c) * (NB * NB);
    };
    if (threadIdx.x < 4) {  // a lane per wait: their polls overlap
      const int wc = rec->wait[threadIdx.x][0], wval = rec->wait[threadIdx.x][1];
      if (wval > 0 && !dag_wait(B.ctr + wc, wval, head + 2))
        atomicCAS((unsigned long long*)B.info, 0ull, (unsigned long long)(int64_t)DL_INFO_TIMEOUT);
    }
    __syncthreads();
    int fk = -1;  // tile to factor, staged in S0
    switch (t.type) {
      case dag::T_F: {
        double va[DPER];
        tile_regs<true>(tile(B.A, t.k, t.k), ld, va);
        regs_to_cols(va, S0);
        __syncthreads();
        fk = t.k;
        break;
      }
      case dag::T_C: {
        // S(k+1, k), then U(k+1, k+1, k) and F(k+1) on the tiles in LDS
        const int k = t.k, k1 = t.k + 1;
        double vg[DPER], va[DPER], dpre[4];
        tile_regs<true>(tile(B.A, k, k), ld, vg);    // G_kk
        tile_regs<true>(tile(B.A, k1, k), ld, va);   // A(k+1, k)
        double* Ad = tile(B.A, k1, k1);               // A(k+1, k+1), final but for U(., ., k)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) dpre[rg] = cload(&Ad[(q0 + lr) + (int64_t)(p0 + lk + 4 * rg) * ld]);
        regs_to_cols(vg, S1);
        regs_to_cols(va, S0);
        __syncthreads();
        v4d a0 = {0.0, 0.0, 0.0, 0.0};
        mfma1_k64(S1, p0, S0, q0, a0, p0 + 16);  // L(m = q0 + lr, c = p0 + lk + 4r)
        double* Lo = tileL(k1, k);
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          cstore(&Lo[(q0 + lr) + (int64_t)(p0 + lk + 4 * rg) * NB], a0[rg]);
          S2[(p0 + lk + 4 * rg) * LDL + q0 + lr] = a0[rg];  // S2[c][m] = L(m, c)
        }
        __syncthreads();
        v4d u0 = {0.0, 0.0, 0.0, 0.0};
        mfma1_k64(S2, p0, S2, q0, u0);  // (L L^T)(m = q0 + lr, n = p0 + lk + 4r)
        // the updated tile, column-major in S0 (read no more since the barrier)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) S0[(p0 + lk + 4 * rg) * LDL + q0 + lr] = dpre[rg] - u0[rg];
        // L(k+1, k) published once every lane's stores are complete (their
        // latency overlaps the update above)
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (threadIdx.x == 0) dag_store(B.ctr + rec->mid[0], rec->mid[1]);
        fk = k1;
        break;
      }
      case dag::T_S: {
        // L(i, k) = A(i, k) G_kk^T: S1[q][r] = G(r, q), S0[c][m] = A(m, c)
        double vg[DPER], va[DPER];
        tile_regs<true>(tile(B.A, t.k, t.k), ld, vg);
        tile_regs<true>(tile(B.A, t.i, t.k), ld, va);
        regs_to_cols(vg, S1);
        regs_to_cols(va, S0);
        __syncthreads();
        v4d a0 = {0.0, 0.0, 0.0, 0.0};
        mfma1_k64(S1, p0, S0, q0, a0, p0 + 16);  // L(m = q0 + lr, c = p0 + lk + 4r)
        double* Lo = tileL(t.i, t.k);
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) cstore(&Lo[(q0 + lr) + (int64_t)(p0 + lk + 4 * rg) * NB], a0[rg]);
        break;
      }
      case dag::T_U: {
        // A(i, k) -= L(i, j) L(k, j)^T for n j's, the next one's tiles in flight
        const bool diag = t.i == t.k;
        double vp[DPER], vq[DPER], cpre[4];
        tile_regs<false>(tileL(t.i, t.j), NB, vp);
        if (!diag) tile_regs<false>(tileL(t.k, t.j), NB, vq);
        double* C = tile(B.A, t.i, t.k);
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) cpre[rg] = cload(&C[(q0 + lr) + (int64_t)(p0 + lk + 4 * rg) * ld]);
        regs_to_cols(vp, S0);
        if (!diag) regs_to_cols(vq, S1);
#pragma unroll 1
        for (int q = 0; q < t.n; ++q) {
          double* X = pool + (q & 1) * 2 * TILE_LDS;
          double* Xn = pool + (~q & 1) * 2 * TILE_LDS;
          if (q + 1 < t.n) {
            tile_regs<false>(tileL(t.i, t.j + q + 1), NB, vp);
            if (!diag) tile_regs<false>(tileL(t.k, t.j + q + 1), NB, vq);
          }
          __syncthreads();
          // rounded like a task of its own
          v4d u0 = {0.0, 0.0, 0.0, 0.0};
          mfma1_k64(diag ? X : X + TILE_LDS, p0, X, q0, u0);  // update(m = q0 + lr, n = p0 + lk + 4r)
#pragma unroll
          for (int rg = 0; rg < 4; ++rg) cpre[rg] -= u0[rg];
          if (q + 1 < t.n) {
            regs_to_cols(vp, Xn);
            if (!diag) regs_to_cols(vq, Xn + TILE_LDS);
          }
        }
#pragma unroll
        for (int rg = 0; rg < 4; ++rg)
          cstore(&C[(q0 + lr) + (int64_t)(p0 + lk + 4 * rg) * ld], cpre[rg]);
        break;
      }
      case dag::T_A:
      case dag::T_R: {
        // A(r, c, m): S(r, c) (+)= L(r, m) G(m, c);
        // R(j, c):    t = S(j, c) + L(j, j-1) G(j-1, c), G(j, c) = -G_jj t
        const bool row = t.type == dag::T_R;
        const int r = t.i, c = t.k, m = row ? t.i - 1 : t.j, n = row ? 1 : t.n;
        double* Sd = B.stage + ((int64_t)r * (r - 1) / 2 + c) * (NB * NB);
        const bool acc = row ? (r - 1 > c) : (m > c);
        double prev[4] = {0.0, 0.0, 0.0, 0.0};
        if (acc) {
#pragma unroll
          for (int rg = 0; rg < 4; ++rg) prev[rg] = cload(&Sd[(q0 + lr) + (p0 + lk + 4 * rg) * NB]);
        }
        double vy[DPER], vx[DPER], vg[DPER];
        tile_regs<false>(tileL(r, m), NB, vy);  // Y = L(r, m)
        tile_regs<true>(tile(B.A, m, c), ld, vx);   // X = G(m, c)
        if (row) tile_regs<true>(tile(B.A, r, r), ld, vg);  // G_jj, for the second product
        regs_to_cols(vy, S0);
        regs_to_rows(vx, S1);
        v4d tv = {prev[0], prev[1], prev[2], prev[3]};
#pragma unroll 1
        for (int q = 0; q < n; ++q) {
          double* X = pool + (q & 1) * 2 * TILE_LDS;
          double* Xn = pool + (~q & 1) * 2 * TILE_LDS;
          if (q + 1 < n) {
            tile_regs<false>(tileL(r, m + q + 1), NB, vy);
            tile_regs<true>(tile(B.A, m + q + 1, c), ld, vx);
          }
          __syncthreads();
          mfma1_k64(X + TILE_LDS, p0, X, q0, tv);  // (Y X)(q0 + lr, p0 + lk + 4r)
          if (q + 1 < n) {
            regs_to_cols(vy, Xn);
            regs_to_rows(vx, Xn + TILE_LDS);
          }
        }
        if (!row) {
#pragma unroll
          for (int rg = 0; rg < 4; ++rg) cstore(&Sd[(q0 + lr) + (p0 + lk + 4 * rg) * NB], tv[rg]);
          break;
        }
        __syncthreads();  // S0, S1 are read no more
        regs_to_cols(vg, S0);  // G_jj
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) S1[(q0 + lr) * LDL + p0 + lk + 4 * rg] = tv[rg];
        __syncthreads();
        v4d g = {0.0, 0.0, 0.0, 0.0};
        mfma1_k64(S1, p0, S0, q0, g, q0 + 16);  // G_jj is lower triangular
        double* dst = tile(B.A, r, c);
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) cstore(&dst[(q0 + lr) + (int64_t)(p0 + lk + 4 * rg) * ld], -g[rg]);
        break;
      }
    }
    if (fk >= 0)
      potrf_body<true>(nullptr, 0, S0, S2, tile(B.A, fk, fk), ld, nullptr,
                       B.logdiag + (int64_t)fk * NB, B.info, B.row0 + (int64_t)fk * NB, 1);
    // every lane's stores complete before the counter is set
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
      dag_store(B.ctr + rec->set[0], rec->set[1]);
      s_task = atomicAdd(head, 1);
    }
    __syncthreads();
  }
  // the last workgroup out (every task is then complete) zeroes the
  // counters and the head for the next launch
  if (threadIdx.x == 0) s_last = atomicAdd(head + 1, 1) == (int)gridDim.x - 1;
  __syncthreads();
  if (s_last) {
    for (int b = 0; b < nblocks; ++b) {
      const int64_t nc = dag::counters_per_block(blocks[b].nbk);
      for (int64_t i = threadIdx.x; i < nc; i += POTRF_NT) dag_store(blocks[b].ctr + i, 0);
    }
    if (threadIdx.x == 0) {
      dag_store(head, 0);
      dag_store(head + 1, 0);
      dag_store(head + 2, 0);
    }
  }
}

hipError_t launch_dag_chol(const DagTask* tasks, int ntask, const DagBlock* blocks,
                           int nblocks, int32_t* head, int workers, hipStream_t s) {
  if (ntask <= 0 || nblocks <= 0 || workers <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_dag_chol, dim3(workers), dim3(POTRF_NT), 0, s, tasks, ntask, blocks,
                     nblocks, head);
  return hipGetLastError();
}

// Batched element-wise jobs: grid (blocks, jobs).
__global__ __launch_bounds__(256) void k_misc(const MiscJob* __restrict__ jobs) {
  const MiscJob J = jobs[blockIdx.y];
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  switch (J.kind) {
    case MJ_FILL:
      for (int64_t i = i0; i < J.n; i += stride) J.dst[i] = J.v;
      break;
    case MJ_COPY:
      for (int64_t i = i0; i < J.n; i += stride) J.dst[i] = J.src[i];
      break;
    case MJ_ZERO_I64:
      for (int64_t i = i0; i < J.n; i += stride) ((int64_t*)J.dst)[i] = 0;
      break;
    case MJ_DIAG:
      for (int64_t i = i0; i < J.n; i += stride) J.dst[i] = J.src[i * (J.lds + 1)];
      break;
    case MJ_COPY2D: {
      const int64_t tot = (int64_t)J.rows * J.cols;
      for (int64_t i = i0; i < tot; i += stride) {
        const int64_t r = i % J.rows, c = i / J.rows;
        J.dst[r + c * J.ldd] = J.src[r + c * J.lds];
      }
      break;
    }
    case MJ_COPY2D_F32: {
      const float* src32 = (const float*)J.src;
      const int64_t tot = (int64_t)J.rows * J.cols;
      for (int64_t i = i0; i < tot; i += stride) {
        const int64_t r = i % J.rows, c = i / J.rows;
        J.dst[r + c * J.ldd] = (double)src32[r + c * J.lds];
      }
      break;
    }
    case MJ_AXPY:
      for (int64_t i = i0; i < J.n; i += stride) J.dst[i] += J.src[i];
      break;
    case MJ_AXPY_UNCONV:
      if (!(J.norms[0] <= J.tol2[0] * J.norms[1]))
        for (int64_t i = i0; i < J.n; i += stride) J.dst[i] += J.src[i];
      break;
    case MJ_COPY2D_TO_F32: {
      float* dst32 = (float*)J.dst;
      const int64_t tot = (int64_t)J.rows * J.cols;
      for (int64_t i = i0; i < tot; i += stride) {
        const int64_t r = i % J.rows, c = i / J.rows;
        dst32[r + c * J.ldd] = (float)J.src[r + c * J.lds];
      }
      break;
    }
    case MJ_COPY2D_LOWER: {
      const int64_t tot = (int64_t)J.rows * J.cols;
      for (int64_t i = i0; i < tot; i += stride) {
        const int64_t r = i % J.rows, c = i / J.rows;
        if (r >= c) J.dst[r + c * J.ldd] = J.src[r + c * J.lds];
      }
      break;
    }
    case MJ_ZERO_UPPER_TILES: {
      const int64_t tot = (int64_t)J.rows * J.rows;
      for (int64_t i = i0; i < tot; i += stride) {
        const int64_t r = i % J.rows, c = i / J.rows;
        if ((r >> 6) < (c >> 6)) J.dst[r + c * J.ldd] = 0.0;
      }
      break;
    }
  }
}

hipError_t launch_misc(const MiscJob* jobs, int count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_misc, dim3(256, count), dim3(256), 0, s, jobs);
  return hipGetLastError();
}

// Deterministic sums: block b of job j reduces a fixed contiguous range with
// a fixed tree; the job's block partials are then reduced in index order.
__device__ __forceinline__ double block_sum_256(double v, double* sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (t < s) sh[t] += sh[t + s];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

__global__ __launch_bounds__(256) void k_sum_partial(const SumJob* __restrict__ jobs) {
  __shared__ double sh[256];
  const SumJob J = jobs[blockIdx.y];
  const int64_t per = (J.n + SUM_BLOCKS - 1) / SUM_BLOCKS;
  const int64_t b0 = (int64_t)blockIdx.x * per;
  const int64_t b1 = min(J.n, b0 + per);
  double acc = 0.0;
  for (int64_t i = b0 + threadIdx.x; i < b1; i += 256) acc += J.src[i];
  const double v = block_sum_256(acc, sh);
  if (threadIdx.x == 0) J.partial[blockIdx.x] = v;
}

__global__ __launch_bounds__(256) void k_sum_final(const SumJob* __restrict__ jobs) {
  __shared__ double sh[256];
  const SumJob J = jobs[blockIdx.x];
  double acc = 0.0;
  for (int i = threadIdx.x; i < SUM_BLOCKS; i += 256) acc += J.partial[i];
  const double v = block_sum_256(acc, sh);
  double acc2 = 0.0;
  if (J.src2)
    for (int64_t i = threadIdx.x; i < J.n2; i += 256) acc2 += J.src2[i];
  const double v2 = block_sum_256(acc2, sh);
  if (threadIdx.x == 0) {
    double r = J.scale * v;
    if (J.src2) r += J.scale2 * v2;
    if (J.add) r += J.add[0];
    J.dst[0] = r;
  }
}

hipError_t launch_sums(const SumJob* jobs, int count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_sum_partial, dim3(SUM_BLOCKS, count), dim3(256), 0, s, jobs);
  hipLaunchKernelGGL(k_sum_final, dim3(count), dim3(256), 0, s, jobs);
  return hipGetLastError();
}

}  // namespace dl
