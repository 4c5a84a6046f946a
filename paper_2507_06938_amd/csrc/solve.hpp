#pragma once
#include "common.hpp"

#define DL_GEMV_FN __host__ __device__ inline
#include "gemv_index.hpp"

namespace dl {

constexpr int SOLVE_RHS = 4;  // right-hand sides of one pass over the factor

// out = beta*base + alpha*A*x, rows [0, split) -> out1/base1 and rows
// [split, M) -> out2/base2 (split < 0: all rows to out1), for the launch's
// right-hand sides r: x + r sx, base1 + r sb1, out1 + r so1, base2 and out2 +
// r s2.  `partial` holds GEMV_KS * nrhs * M doubles and `cnt` one zero per 128
// rows, both private to this job's launch.  M, K, lda, split and the vectors'
// strides are multiples of 64 (16-byte loads).
struct GemvN {
  int M, K;
  const double* A;
  int64_t lda;
  const double* x;
  int tri;
  double alpha, beta;
  int split;
  const double* base1;
  double* out1;
  const double* base2;
  double* out2;
  double* partial;
  int32_t* cnt;
  int a32;  // A stored in FP32
  int64_t sx, sb1, so1, s2;
  Band band;  // of A's rows (period 0: dense)
};

// y = beta*base + alpha*A^T*x with x = [x1 (rows < split); x2], for the
// launch's right-hand sides r: x1 + r sx1, x2 + r sx2, base + r sb, y + r sy.
// The same alignment as above; N is a multiple of 8.
struct GemvT {
  int M, N;
  const double* A;
  int64_t lda;
  const double* x1;
  int split;
  const double* x2;
  int tri;
  double alpha, beta;
  const double* base;
  double* y;
  int a32;  // A stored in FP32
  int64_t sx1, sx2, sb, sy;
  Band band;  // of A's rows (period 0: dense)
};

// Batched launches over job arrays in device memory; max_M / max_K / max_N bound
// the grid over all jobs; nrhs: 1 or SOLVE_RHS.
hipError_t launch_gemv_n(const GemvN* jobs_dev, int count, int max_M, int max_K, int nrhs,
                         hipStream_t s);
hipError_t launch_gemv_t(const GemvT* jobs_dev, int count, int max_N, int nrhs,
                         hipStream_t s);

}  // namespace dl
