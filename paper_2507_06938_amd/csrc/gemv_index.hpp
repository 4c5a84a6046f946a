// Column slices of the matrix-vector products and the columns their waves load.
// No HIP types: the kernel (solve.hip) and a CPU test that walks over every block
// size use the same functions.  A HIP translation unit defines DL_GEMV_FN as
// __host__ __device__ inline before including this header.
#pragma once

#ifndef DL_GEMV_FN
#define DL_GEMV_FN inline
#endif

namespace dl {

constexpr int GEMV_KS = 32;      // most column slices of a matrix-vector product
constexpr int GEMV_STAGE = 128;  // columns of a slice whose x is staged at a time

// Columns of a slice of K (a multiple of 64) columns: 64, or what makes GEMV_KS slices
// of them.  One slice up to 256 columns saves the hand-over to the last workgroup but
// not the time of three more rounds of loads: a solve of 20 blocks of 256 rows took
// 477 us with it, 342 without, of 192 rows 410 / 323, of 128 rows 327 / 316.
DL_GEMV_FN constexpr int gemv_slice_len(int K) {
  return K <= 64 * GEMV_KS ? 64 : (K + GEMV_KS - 1) / GEMV_KS;
}

// The column of a stage of nb that a wave loads for column c of its share: c, or
// the first one when there is none left (the value is not used).  Beyond 2048
// columns a slice may end in a stage of fewer columns than there are waves.
DL_GEMV_FN constexpr int gemv_column(int c, int nb) { return c < nb ? c : 0; }

}  // namespace dl
