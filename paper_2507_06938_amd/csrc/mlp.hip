// Surrogate network kernels: a multi-layer perceptron x -> SiLU(W1 x + b1)
// -> ... -> W_L h + b_L trained on the GPU.  Weights are kept in FP32
// (master copy, Adam moments); every matrix product rounds both operands to
// bfloat16 (round to nearest even) and accumulates in FP32 on the matrix cores.
//
// The network of the surrogate (256 wide, batches of tens to thousands of
// rows) is bound by latency: a product of it takes a microsecond, a launch and
// the first loads of it several.  So a forward pass is one launch (k_mlp_fwd:
// a workgroup takes 16 rows through all layers, activations in LDS), a backward
// pass two (k_mlp_bwd_rows: the same for d loss / d Z; k_mlp_bwd_weights: the
// weight and bias gradients of all layers).  A training step on 930 rows of
// the 15-256-256-256-1 network went from 1190 to 57 us, of which 644 us were
// serial column sums and 530 us products with one 16-deep chunk in flight; the
// gradient at one point from 150 to 37 us.  What is left of the forward launch
// (21 us for one row, 25 for 930) is one compute unit's fetch of the weights
// (540 KB) beyond its XCD's L2; staging whole rows of W through LDS, prefetching
// the next layer's block in registers (spills) and the arguments in device
// memory did not shorten it.  Wide layers and large batches take one launch per
// product where that is ahead (whole_fwd, whole_bwd), as do networks wider than
// MLP_WMAX or deeper than MLP_LMAX (their rows do not fit LDS, their layers not the
// kernels' arguments).
#include <math.h>
#include <stdint.h>

#include <new>
#include <vector>

#include "engine.hpp"

namespace dl {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;  // NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}

// C[m][n] = act(alpha * sum_k A(m,k) B(n,k) + bias[n]) (+ beta * C_old),
// A(m,k) = A[m*sam + k*sak], B(n,k) = B[n*sbn + k*sbk] (FP32, any strides),
// Z (pre-activation) and H (output) row-major with leading dims ldz / ldh.
// One workgroup (4 waves) per 64x64 tile; the k loop stages 16-deep bf16
// chunks in LDS.  MFMA operands: op(B) as "A" and op(A) as "B", so the
// accumulator holds C^T and lane l, register r is C[m0 + l%16][n0 + 4(l/16)
// + r] within its 16x16 block.
struct LinJob {
  int M, N, K;
  const float* A;
  int64_t sam, sak;
  const float* B;
  int64_t sbn, sbk;
  const float* bias;
  float alpha, beta;
  float* Z;
  int64_t ldz;
  float* H;
  int64_t ldh;
  int act;  // 0 none, 1 SiLU
};

__global__ __launch_bounds__(256) void k_mlp_linear(LinJob J) {
  __shared__ unsigned short As[64][16 + 4];
  __shared__ unsigned short Bs[64][16 + 4];
  const int tid = threadIdx.x;
  const int m0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  const int l16 = lane & 15, lg = lane >> 4;
  v4f acc[2][2];
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < 2; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < J.K; k0 += 16) {
    for (int e = tid; e < 64 * 16; e += 256) {
      const int r = e >> 4, kk = e & 15;
      const int k = k0 + kk;
      const int m = m0 + r, n = n0 + r;
      const float a = (m < J.M && k < J.K) ? J.A[(int64_t)m * J.sam + (int64_t)k * J.sak] : 0.f;
      const float b = (n < J.N && k < J.K) ? J.B[(int64_t)n * J.sbn + (int64_t)k * J.sbk] : 0.f;
      As[r][kk] = f2bf(a);
      Bs[r][kk] = f2bf(b);
    }
    __syncthreads();
    v4s fa[2], fb[2];
    for (int i = 0; i < 2; ++i) {
      const unsigned short* p = &As[wm * 32 + i * 16 + l16][4 * lg];
      fa[i] = (v4s){(short)p[0], (short)p[1], (short)p[2], (short)p[3]};
    }
    for (int j = 0; j < 2; ++j) {
      const unsigned short* p = &Bs[wn * 32 + j * 16 + l16][4 * lg];
      fb[j] = (v4s){(short)p[0], (short)p[1], (short)p[2], (short)p[3]};
    }
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fb[j], fa[i], acc[i][j], 0, 0, 0);
    __syncthreads();
  }
  for (int i = 0; i < 2; ++i) {
    const int m = m0 + wm * 32 + i * 16 + l16;
    if (m >= J.M) continue;
    for (int j = 0; j < 2; ++j)
      for (int r = 0; r < 4; ++r) {
        const int n = n0 + wn * 32 + j * 16 + 4 * lg + r;
        if (n >= J.N) continue;
        float z = J.alpha * acc[i][j][r] + (J.bias ? J.bias[n] : 0.f);
        if (J.Z) J.Z[(int64_t)m * J.ldz + n] = z;
        float h = z;
        if (J.act == 1) h = z / (1.f + expf(-z));
        if (J.H) {
          float* p = J.H + (int64_t)m * J.ldh + n;
          *p = (J.beta != 0.f) ? h + J.beta * (*p) : h;
        }
      }
  }
}

// ---- whole passes ----------------------------------------------------------------------
constexpr int MLP_LMAX = 16;    // layers
constexpr int MLP_WMAX = 2048;  // widest layer: 2 x 16 rows of bfloat16 in LDS
constexpr int MLP_ROWS = 16;    // rows of a workgroup
constexpr int MLP_NT = 1024;
constexpr int MLP_PAD = 8;      // row padding in LDS (16 bytes: rows start 4 banks apart)

struct MlpArgs {
  int L, ld;                    // layers, LDS row length
  int size[MLP_LMAX + 1];
  int64_t woff[MLP_LMAX], boff[MLP_LMAX];
  const float* w;
  float* Z[MLP_LMAX];           // pre-activations
  float* H[MLP_LMAX];           // layer inputs
  float* G[MLP_LMAX];           // d loss / d Z (null for the last layer: dy)
  float* yhat;
};

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v8f __attribute__((ext_vector_type(8)));

// acc[m][n] += sum_k A(m, k) B(n, k) over 32 k (v_mfma_f32_16x16x32_bf16: lane
// l supplies A(l % 16, 8 (l / 16) + j) and B(l % 16, 8 (l / 16) + j), j < 8;
// its register r receives acc(4 (l / 16) + r, l % 16))
__device__ __forceinline__ v4f mma32(v8bf a, v8bf b, v4f acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
}

// Zero the columns [w, w rounded up to 32) of 16 staged rows.
__device__ __forceinline__ void zero_tail(__bf16* act, int ld, int w) {
  const int m = threadIdx.x >> 5, c = w + (threadIdx.x & 31);
  if (m < MLP_ROWS && c < ((w + 31) & ~31)) act[m * ld + c] = (__bf16)0.f;
}

// One 16-column block's product of the staged rows (ar: row l % 16, from k = 8
// (l / 16)) with a layer's weights.  256 k at a time all weights of the block
// are loaded before the first is used: their latency is what a layer costs.
// The code is kept short: with one workgroup a pass its first fetch into the
// instruction cache is part of the time.
// col_product: operand column c's value for k at p[k * sk] (p already at this
// lane's column and first k), 16 consecutive columns in memory.
__device__ __forceinline__ v4f col_product(const __bf16* ar, const float* __restrict__ p,
                                           int64_t sk, int K, int lk, int k0 = 0,
                                           v4f acc = (v4f){0.f, 0.f, 0.f, 0.f}) {
  if (sk > 1) {
#pragma unroll 1
    for (; k0 + 256 <= K; k0 += 256) {
      v8f x[8];
#pragma unroll
      for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int j = 0; j < 8; ++j) x[s][j] = p[(k0 + 32 * s + j) * sk];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < 8; ++s)
        acc = mma32(*(const v8bf*)(ar + k0 + 32 * s), __builtin_convertvector(x[s], v8bf), acc);
    }
  }
#pragma unroll 1
  for (; k0 < K; k0 += 32) {
    v8f x;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = k0 + 8 * lk + j;
      const float v = p[(int64_t)(min(k, K - 1) - 8 * lk) * sk];
      x[j] = k < K ? v : 0.f;
    }
    acc = mma32(*(const v8bf*)(ar + k0), __builtin_convertvector(x, v8bf), acc);
  }
  return acc;
}

// row_product: operand row l % 16 is the row of W at p (already at this lane's
// first k); vec: K and p allow 16-byte loads.
__device__ __forceinline__ v4f row_product(const __bf16* ar, const float* __restrict__ p, int K,
                                           bool vec, int lk) {
  v4f acc = {0.f, 0.f, 0.f, 0.f};
  int k0 = 0;
#pragma unroll 1
  for (; vec && k0 + 256 <= K; k0 += 256) {
    v4f x[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) x[s] = *(const v4f*)(p + k0 + 32 * (s >> 1) + 4 * (s & 1));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const v4f a = x[2 * s], b = x[2 * s + 1];
      const v8f v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
      acc = mma32(*(const v8bf*)(ar + k0 + 32 * s), __builtin_convertvector(v, v8bf), acc);
    }
  }
  return col_product(ar, p, 1, K, lk, k0, acc);
}

// A workgroup takes rows 16 blockIdx.x .. through all layers; wave w computes
// the 16-column blocks w, w + 16, ..
__global__ __launch_bounds__(MLP_NT) void k_mlp_fwd(MlpArgs N, const float* __restrict__ X, int n,
                                                    float* __restrict__ yhat) {
  extern __shared__ __attribute__((aligned(16))) __bf16 lds[];
  const int ld = N.ld, r0 = blockIdx.x * MLP_ROWS;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  __bf16* cur = lds;
  __bf16* nxt = lds + MLP_ROWS * ld;
  {
    const int in = N.size[0];
    zero_tail(cur, ld, in);
    const bool ok = r0 + wave < n;  // wave w stages row w
    const int64_t row = (int64_t)(r0 + wave) * in;
#pragma unroll 1
    for (int k = lane; k < in; k += 64) {
      const float v = ok ? X[row + k] : 0.f;
      if (ok) N.H[0][row + k] = v;
      cur[wave * ld + k] = (__bf16)v;
    }
  }
  __syncthreads();
#pragma unroll 1
  for (int k = 0; k < N.L; ++k) {
    const int in = N.size[k], out = N.size[k + 1];
    const bool last = k + 1 == N.L;
    const float* W = N.w + N.woff[k];
    const float* bias = N.w + N.boff[k];
    const bool vec = (in & 3) == 0 && (reinterpret_cast<uintptr_t>(W) & 15) == 0;
    if (!last) zero_tail(nxt, ld, out);
#pragma unroll 1
    for (int cb = wave; cb * 16 < out; cb += MLP_NT / 64) {
      const int o = cb * 16 + lr;
      const bool ok = o < out;
      const float b = bias[ok ? o : 0];
      const v4f acc = row_product(cur + lr * ld + 8 * lk,
                                  W + (int64_t)(ok ? o : 0) * in + 8 * lk, in, vec, lk);
      if (!ok) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 4 * lk + r;
        const int64_t at = (int64_t)(r0 + m) * out + o;
        const float z = acc[r] + b;
        const float h = last ? z : z / (1.f + expf(-z));
        if (!last) nxt[m * ld + o] = (__bf16)h;
        if (r0 + m >= n) continue;
        N.Z[k][at] = z;
        if (!last) {
          N.H[k + 1][at] = h;
        } else {
          N.yhat[at] = h;
          if (yhat) yhat[at] = h;
        }
      }
    }
    __syncthreads();
    __bf16* t = cur;
    cur = nxt;
    nxt = t;
  }
}

// d loss / d Z of every layer (and d loss / d X) for rows 16 blockIdx.x ..:
// G_{k-1} = (G_k W_k) SiLU'(Z_{k-1}).
__global__ __launch_bounds__(MLP_NT) void k_mlp_bwd_rows(MlpArgs N, const float* __restrict__ dy,
                                                         int n, float* __restrict__ dX) {
  extern __shared__ __attribute__((aligned(16))) __bf16 lds[];
  const int ld = N.ld, r0 = blockIdx.x * MLP_ROWS;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  __bf16* cur = lds;
  __bf16* nxt = lds + MLP_ROWS * ld;
  zero_tail(cur, ld, 1);
  if (threadIdx.x < MLP_ROWS)
    cur[threadIdx.x * ld] = (__bf16)(r0 + (int)threadIdx.x < n ? dy[r0 + threadIdx.x] : 0.f);
  __syncthreads();
#pragma unroll 1
  for (int k = N.L - 1; k >= (dX ? 0 : 1); --k) {
    const int in = N.size[k], out = N.size[k + 1];
    const float* W = N.w + N.woff[k];
    if (k > 0) zero_tail(nxt, ld, in);
#pragma unroll 1
    for (int cb = wave; cb * 16 < in; cb += MLP_NT / 64) {
      const int i = cb * 16 + lr;
      const bool ok = i < in;
      const float* wc = W + (ok ? i : 0) + (int64_t)(8 * lk) * in;
      const __bf16* ar = cur + lr * ld + 8 * lk;
      float z[4] = {0.f, 0.f, 0.f, 0.f};
      if (k > 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (ok && r0 + 4 * lk + r < n) z[r] = N.Z[k - 1][(int64_t)(r0 + 4 * lk + r) * in + i];
      }
      const v4f acc = col_product(ar, wc, in, out, lk);
      if (!ok) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 4 * lk + r;
        const int64_t at = (int64_t)(r0 + m) * in + i;
        if (k > 0) {
          const float sg = 1.f / (1.f + expf(-z[r]));
          const float g = acc[r] * sg * (1.f + z[r] * (1.f - sg));
          nxt[m * ld + i] = (__bf16)(r0 + m < n ? g : 0.f);
          if (r0 + m < n) N.G[k - 1][at] = g;
        } else if (r0 + m < n) {
          dX[at] = acc[r];
        }
      }
    }
    __syncthreads();
    __bf16* t = cur;
    cur = nxt;
    nxt = t;
  }
}

// dW_k = G_k^T H_k and db_k = column sums of G_k, all layers: one 32 x 32 tile
// of one dW_k per workgroup (`first[k]`: the first workgroup of layer k), its
// 16 waves taking every 16th 32 rows and summed in wave order (the rows of a
// 930-row batch are then in flight at once; with 4 waves the launch took 32 us).
// The rows are read straight into the MFMA operands (lanes along the columns).
struct MlpTiles {
  int first[MLP_LMAX + 1];
};
__global__ __launch_bounds__(MLP_NT) void k_mlp_bwd_weights(MlpArgs N, MlpTiles T,
                                                         const float* __restrict__ dy, int n,
                                                         float* __restrict__ grads) {
  constexpr int NW = MLP_NT / 64;
  __shared__ float sum[NW][32][33];
  __shared__ float bsum[NW][32];
  int k = 0;
  while ((int)blockIdx.x >= T.first[k + 1]) ++k;
  const int in = N.size[k], out = N.size[k + 1];
  const int ti = (in + 31) / 32;
  const int t = blockIdx.x - T.first[k];
  const int o0 = 32 * (t / ti), i0 = 32 * (t % ti);
  const float* G = N.G[k] ? N.G[k] : dy;
  const float* H = N.H[k];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  int oc[2], ic[2];
  bool oo[2], io[2];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    oc[b] = o0 + 16 * b + lr;
    ic[b] = i0 + 16 * b + lr;
    oo[b] = oc[b] < out;
    io[b] = ic[b] < in;
    if (!oo[b]) oc[b] = 0;
    if (!io[b]) ic[b] = 0;
  }
  v4f acc[2][2];
  float bs[2] = {0.f, 0.f};
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
  for (int m0 = 32 * wave; m0 < n; m0 += 32 * NW) {
    v8f g[2], h[2];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int m = m0 + 8 * lk + j;
      const bool ok = m < n;
      const int64_t mm = ok ? m : 0;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const float gv = G[mm * out + oc[b]], hv = H[mm * in + ic[b]];
        g[b][j] = ok && oo[b] ? gv : 0.f;
        h[b][j] = ok && io[b] ? hv : 0.f;
      }
    }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int j = 0; j < 8; ++j) bs[b] += g[b][j];
    v8bf gb[2], hb[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      gb[b] = __builtin_convertvector(g[b], v8bf);
      hb[b] = __builtin_convertvector(h[b], v8bf);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[a][b] = mma32(gb[a], hb[b], acc[a][b]);
  }
#pragma unroll
  for (int a = 0; a < 2; ++a) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[wave][16 * a + 4 * lk + r][16 * b + lr] = acc[a][b][r];
    bs[a] += __shfl_xor(bs[a], 16, 64);
    bs[a] += __shfl_xor(bs[a], 32, 64);
    if (lk == 0) bsum[wave][16 * a + lr] = bs[a];
  }
  __syncthreads();
  {
    const int a = threadIdx.x >> 5, b = threadIdx.x & 31;
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < NW; ++q) v += sum[q][a][b];
    if (o0 + a < out && i0 + b < in) grads[N.woff[k] + (int64_t)(o0 + a) * in + i0 + b] = v;
  }
  if (i0 == 0 && threadIdx.x < 32 && o0 + (int)threadIdx.x < out) {
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < NW; ++q) v += bsum[q][threadIdx.x];
    grads[N.boff[k] + o0 + threadIdx.x] = v;
  }
}

static hipError_t linear(const LinJob& J, hipStream_t s) {
  if (J.M <= 0 || J.N <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mlp_linear, dim3((J.M + 63) / 64, (J.N + 63) / 64), dim3(256),
                     0, s, J);
  return hipGetLastError();
}

// dZ = dH * SiLU'(Z)
__global__ void k_silu_bwd(int64_t n, const float* dH, const float* Z, float* dZ) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float z = Z[i];
    const float sg = 1.f / (1.f + expf(-z));
    dZ[i] = dH[i] * sg * (1.f + z * (1.f - sg));
  }
}

// out[n] = sum over rows m of X[m*ld + n] (fixed order per column)
__global__ void k_colsum(int M, int N, const float* X, int64_t ld, float* out) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  float s = 0.f;
  for (int m = 0; m < M; ++m) s += X[(int64_t)m * ld + n];
  out[n] = s;
}

// dy = 2 (yhat - y) / n; loss = mean (yhat - y)^2 (one block, fixed tree)
__global__ void k_mse(int n, const float* yhat, const float* y, float* dy, float* loss) {
  __shared__ float sh[256];
  float acc = 0.f;
  for (int i = threadIdx.x; i < n; i += 256) {
    const float r = yhat[i] - y[i];
    dy[i] = 2.f * r / (float)n;
    acc += r * r;
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0 && loss) loss[0] = sh[0] / (float)n;
}

// Adam (Kingma & Ba) on a flat parameter vector.
__global__ void k_adam(int64_t n, float* w, const float* g, float* m, float* v,
                       float lr, float b1, float b2, float eps, float c1, float c2) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

}  // namespace dl

using namespace dl;

struct dl_mlp {
  std::vector<int> sizes;   // in, hidden..., out
  int max_batch = 0;
  int64_t nparam = 0;
  std::vector<int64_t> woff, boff;  // offsets of W_k (out x in, row-major), b_k
  float *w = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;
  std::vector<float*> Z, Hs;  // pre-activations and layer inputs (H[0] = X copy)
  std::vector<float*> G;      // d loss / d Z_k (max_batch x out_k; the last: none)
  bool whole = false;         // whole passes possible (MLP_WMAX, MLP_LMAX)
  int widest = 0;             // most outputs of a layer
  MlpArgs args{};
  MlpTiles tiles{};
  size_t lds = 0;             // bytes of k_mlp_fwd and k_mlp_bwd_rows
  float *yhat = nullptr, *dy = nullptr, *loss = nullptr;
  int step = 0;
  int last_n = 0;
  std::vector<void*> allocs;
};

extern "C" dl_status dl_mlp_create(const int32_t* sizes, int32_t nsizes,
                                   int32_t max_batch, dl_mlp** out) {
  if (!sizes || nsizes < 2 || max_batch <= 0 || !out) return DL_EINVAL;
  for (int k = 0; k < nsizes; ++k)
    if (sizes[k] <= 0) return DL_EINVAL;
  if (sizes[nsizes - 1] != 1) return DL_EINVAL;
  dl_mlp* N = new (std::nothrow) dl_mlp();
  if (!N) return DL_ENOMEM;
  N->sizes.assign(sizes, sizes + nsizes);
  N->max_batch = max_batch;
  int64_t off = 0;
  int wmax = 0;
  for (int k = 0; k + 1 < nsizes; ++k) {
    N->woff.push_back(off);
    off += (int64_t)sizes[k] * sizes[k + 1];
    N->boff.push_back(off);
    off += sizes[k + 1];
  }
  for (int k = 0; k < nsizes; ++k) wmax = std::max(wmax, sizes[k]);
  for (int k = 1; k < nsizes; ++k) N->widest = std::max(N->widest, sizes[k]);
  N->nparam = off;
  dl_status st = DL_OK;
  auto A = [&](size_t bytes, void** p) {
    if (st == DL_OK) st = dev_alloc(N->allocs, bytes, p);
  };
  A(sizeof(float) * off, (void**)&N->w);
  A(sizeof(float) * off, (void**)&N->g);
  A(sizeof(float) * off, (void**)&N->m);
  A(sizeof(float) * off, (void**)&N->v);
  const int L = nsizes - 1;
  N->Z.resize(L);
  N->Hs.resize(L);
  for (int k = 0; k < L; ++k) {
    A(sizeof(float) * (size_t)max_batch * sizes[k + 1], (void**)&N->Z[k]);
    A(sizeof(float) * (size_t)max_batch * sizes[k], (void**)&N->Hs[k]);
  }
  N->G.resize(L);
  for (int k = 0; k < L; ++k)
    A(sizeof(float) * (size_t)max_batch * sizes[k + 1], (void**)&N->G[k]);
  A(sizeof(float) * max_batch, (void**)&N->yhat);
  A(sizeof(float) * max_batch, (void**)&N->dy);
  A(sizeof(float) * 4, (void**)&N->loss);
  if (st == DL_OK &&
      (hipMemset(N->m, 0, sizeof(float) * off) != hipSuccess ||
       hipMemset(N->v, 0, sizeof(float) * off) != hipSuccess))
    st = DL_EHIP;
  N->whole = wmax <= MLP_WMAX && L <= MLP_LMAX;
  if (N->whole && st == DL_OK) {
    MlpArgs& a = N->args;
    a.L = L;
    a.ld = (wmax + 31) / 32 * 32 + MLP_PAD;
    a.w = N->w;
    a.yhat = N->yhat;
    int tiles = 0;
    for (int k = 0; k <= L; ++k) a.size[k] = sizes[k];
    for (int k = 0; k < L; ++k) {
      a.woff[k] = N->woff[k];
      a.boff[k] = N->boff[k];
      a.Z[k] = N->Z[k];
      a.H[k] = N->Hs[k];
      a.G[k] = k + 1 < L ? N->G[k] : nullptr;
      N->tiles.first[k] = tiles;
      tiles += ((sizes[k] + 31) / 32) * ((sizes[k + 1] + 31) / 32);
    }
    N->tiles.first[L] = tiles;
    N->lds = sizeof(__bf16) * 2 * MLP_ROWS * (size_t)a.ld;
    // the limit is the function's, not the network's: always the widest one's
    constexpr int most = sizeof(__bf16) * 2 * MLP_ROWS * (MLP_WMAX + MLP_PAD);
    if (N->lds > 65536)
      for (const void* f : {(const void*)k_mlp_fwd, (const void*)k_mlp_bwd_rows})
        if (st == DL_OK && hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                               most) != hipSuccess)
          st = DL_EHIP;
  }
  if (st != DL_OK) {
    free_all(N->allocs);
    delete N;
    return st;
  }
  *out = N;
  return DL_OK;
}

extern "C" void dl_mlp_destroy(dl_mlp* N) {
  if (!N) return;
  free_all(N->allocs);
  delete N;
}

extern "C" dl_status dl_mlp_params(dl_mlp* N, float** params_dev, float** grads_dev,
                                   int64_t* count) {
  if (!N) return DL_EINVAL;
  if (params_dev) *params_dev = N->w;
  if (grads_dev) *grads_dev = N->g;
  if (count) *count = N->nparam;
  return DL_OK;
}

// Which passes one launch takes, by the widest layer and the rows (us, one launch /
// one per product; networks of three equal hidden layers; every other size between
// lies between).
//
// Forward, a workgroup of 16 waves goes through 16 rows, 256 columns at a time, and
// its time is its own fetch of the weights until 4096 rows fill the card:
//   * up to 512 columns it is always ahead there (1 row 65 / 110, 4096 rows 73 / 172);
//   * wider, the fetch is longer than the launches it saves unless the rows keep the
//     product launches long: 640 columns 1 row 149 / 133, 32 rows 152 / 155; 1024
//     columns 32 rows 240 / 230, 64 rows 240 / 275; 1280 columns 512 rows 368 / 359,
//     1024 rows 368 / 383; 2048 columns 901 / 426 and still behind at 16384 rows;
//   * a round of 256 columns that is not full costs a full one: 896 columns 1024 rows
//     261 / 260, 4096 rows 262 / 319;
//   * from 4096 rows on the 64 x 64 tiles of the product launches read W less often:
//     8192 rows 384 columns 155 / 162, 640 columns 315 / 266; 16384 rows 64 columns
//     46 / 48, 384 columns 298 / 213, 768 columns 565 / 593; 65536 rows 64 columns
//     162 / 91, 256 columns 365 / 374, 512 columns 1075 / 1012.
static bool whole_fwd(const dl_mlp* N, int n) {
  if (!N->whole) return false;
  const int w = N->widest, round = (w + 255) / 256 * 256;
  const bool fills = 10 * w > 9 * round;
  if (n > 16384) return fills && round == 256;
  if (n > 4096) return w <= 64 || (n <= 8192 && w <= 512) || (fills && round <= 768);
  switch (round / 256) {
    case 1: case 2: return true;
    case 3: return fills || n > 16;
    case 4: return n > (fills ? 32 : 1024);
    case 5: return n > (fills ? 512 : 2048);
    case 6: return fills && n > 2048;
    default: return false;
  }
}

// Backward, where the weights' launch sums over rows and the product launches of the
// column sums are serial: behind only where a few rows meet wide layers (1280 columns,
// 1 row 254 / 223, 64 rows 306 / 359; 2048 columns, 1 row 581 / 426, 64 rows 667 / 535,
// 256 rows 650 / 799; with d loss / d X 1280 columns 1 row 257 / 291, 2048 columns 16
// rows 663 / 557, 64 rows 676 / 707).
static bool whole_bwd(const dl_mlp* N, int n, bool dx) {
  const int w = N->widest;
  if (dx) return N->whole && (w <= 1792 || n > 32);
  return N->whole && (w <= 1152 || n > (w > 1664 ? 128 : 32));
}

// Do the n floats at a and the m floats at b share memory?
static bool overlap(const float* a, int64_t n, const float* b, int64_t m) {
  return a && b && a < b + m && b < a + n;
}

extern "C" dl_status mlp_fwd(dl_mlp* N, const float* X, int32_t n, float* yhat,
                             void* stream) {
  if (!N || !X || n <= 0 || n > N->max_batch) return DL_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  if (whole_fwd(N, n)) {
    // outputs over the inputs: a workgroup's would reach rows not yet read
    const bool over = overlap(X, (int64_t)n * N->sizes[0], yhat, n);
    hipLaunchKernelGGL(k_mlp_fwd, dim3((n + MLP_ROWS - 1) / MLP_ROWS), dim3(MLP_NT), N->lds,
                       s, N->args, X, n, over ? nullptr : yhat);
    DL_HIP_CHECK(hipGetLastError());
    if (over)
      DL_HIP_CHECK(hipMemcpyAsync(yhat, N->yhat, sizeof(float) * n, hipMemcpyDeviceToDevice, s));
    N->last_n = n;
    return DL_OK;
  }
  const int L = (int)N->sizes.size() - 1;
  const float* hin = X;
  int64_t ldin = N->sizes[0];
  DL_HIP_CHECK(hipMemcpyAsync(N->Hs[0], X, sizeof(float) * (size_t)n * N->sizes[0],
                              hipMemcpyDeviceToDevice, s));
  hin = N->Hs[0];
  for (int k = 0; k < L; ++k) {
    const int in = N->sizes[k], outw = N->sizes[k + 1];
    LinJob J{};
    J.M = n; J.N = outw; J.K = in;
    J.A = hin; J.sam = ldin; J.sak = 1;
    J.B = N->w + N->woff[k]; J.sbn = in; J.sbk = 1;
    J.bias = N->w + N->boff[k];
    J.alpha = 1.f; J.beta = 0.f;
    J.Z = N->Z[k]; J.ldz = outw;
    const bool lastl = (k + 1 == L);
    J.H = lastl ? N->yhat : N->Hs[k + 1];
    J.ldh = outw;
    J.act = lastl ? 0 : 1;
    DL_HIP_CHECK(linear(J, s));
    hin = J.H;
    ldin = outw;
  }
  if (yhat)
    DL_HIP_CHECK(hipMemcpyAsync(yhat, N->yhat, sizeof(float) * n,
                                hipMemcpyDeviceToDevice, s));
  N->last_n = n;
  return DL_OK;
}

// Backward of the last mlp_fwd: dy (n) -> parameter gradients (overwritten)
// and, when dX != NULL, d(sum dy*yhat)/dX (n x in, row-major).
extern "C" dl_status mlp_bwd(dl_mlp* N, const float* dy, int32_t n, float* dX,
                             void* stream) {
  if (!N || !dy || n != N->last_n) return DL_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  const int L = (int)N->sizes.size() - 1;
  if (whole_bwd(N, n, dX != nullptr)) {
    if (overlap(dy, n, dX, (int64_t)n * N->sizes[0])) {
      // dX over dy, which the last layer's gradients are formed from as well
      DL_HIP_CHECK(hipMemcpyAsync(N->G[L - 1], dy, sizeof(float) * n, hipMemcpyDeviceToDevice,
                                  s));
      dy = N->G[L - 1];
    }
    if (L > 1 || dX) {
      hipLaunchKernelGGL(k_mlp_bwd_rows, dim3((n + MLP_ROWS - 1) / MLP_ROWS), dim3(MLP_NT),
                         N->lds, s, N->args, dy, n, dX);
      DL_HIP_CHECK(hipGetLastError());
    }
    hipLaunchKernelGGL(k_mlp_bwd_weights, dim3(N->tiles.first[L]), dim3(MLP_NT), 0, s, N->args,
                       N->tiles, dy, n, N->g);
    DL_HIP_CHECK(hipGetLastError());
    return DL_OK;
  }
  // g = dL/dZ_k (n x out_k)
  const float* g = dy;
  for (int k = L - 1; k >= 0; --k) {
    const int in = N->sizes[k], outw = N->sizes[k + 1];
    // dW_k = g^T H_k  (outw x in):  C[o][i] = sum_m g[m][o] H[m][i]
    LinJob Jw{};
    Jw.M = outw; Jw.N = in; Jw.K = n;
    Jw.A = g; Jw.sam = 1; Jw.sak = outw;
    Jw.B = N->Hs[k]; Jw.sbn = 1; Jw.sbk = in;
    Jw.alpha = 1.f; Jw.beta = 0.f;
    Jw.H = N->g + N->woff[k]; Jw.ldh = in;
    DL_HIP_CHECK(linear(Jw, s));
    hipLaunchKernelGGL(k_colsum, dim3((outw + 255) / 256), dim3(256), 0, s, n, outw,
                       g, (int64_t)outw, N->g + N->boff[k]);
    DL_HIP_CHECK(hipGetLastError());
    if (k == 0 && !dX) break;
    // dH_k = g W_k  (n x in): C[m][i] = sum_o g[m][o] W[o][i]
    LinJob Jh{};
    Jh.M = n; Jh.N = in; Jh.K = outw;
    Jh.A = g; Jh.sam = outw; Jh.sak = 1;
    Jh.B = N->w + N->woff[k]; Jh.sbn = 1; Jh.sbk = in;
    Jh.alpha = 1.f; Jh.beta = 0.f;
    float* dh = (k == 0) ? dX : N->G[k - 1];
    Jh.H = dh; Jh.ldh = in;
    DL_HIP_CHECK(linear(Jh, s));
    if (k == 0) break;
    // dZ_{k-1} = dH_k * SiLU'(Z_{k-1})
    const int64_t cnt = (int64_t)n * in;
    hipLaunchKernelGGL(k_silu_bwd, dim3((unsigned)std::min<int64_t>(1024, (cnt + 255) / 256)),
                       dim3(256), 0, s, cnt, dh, N->Z[k - 1], dh);
    DL_HIP_CHECK(hipGetLastError());
    g = dh;
  }
  return DL_OK;
}

// dy = 2 (yhat - y)/n from the last forward's output; loss_dev[0] = MSE.
extern "C" dl_status mlp_mse_grad(dl_mlp* N, const float* y, int32_t n, float* dy,
                                  float* loss_dev, void* stream) {
  if (!N || !y || !dy || n != N->last_n) return DL_EINVAL;
  hipLaunchKernelGGL(k_mse, dim3(1), dim3(256), 0, (hipStream_t)stream, n, N->yhat,
                     y, dy, loss_dev);
  DL_HIP_CHECK(hipGetLastError());
  return DL_OK;
}

extern "C" dl_status mlp_adam(dl_mlp* N, float lr, float b1, float b2, float eps,
                              void* stream) {
  if (!N) return DL_EINVAL;
  N->step += 1;
  const float c1 = 1.f - powf(b1, (float)N->step);
  const float c2 = 1.f - powf(b2, (float)N->step);
  hipLaunchKernelGGL(k_adam, dim3(512), dim3(256), 0, (hipStream_t)stream, N->nparam,
                     N->w, N->g, N->m, N->v, lr, b1, b2, eps, c1, c2);
  DL_HIP_CHECK(hipGetLastError());
  return DL_OK;
}
