// The columns that the workgroups of the matrix-vector product load and multiply
// (the loops of gemv_n_body, solve.hip, on csrc/gemv_index.hpp), for every matrix
// size the library accepts: no load outside the columns of the matrix, every
// column multiplied exactly once by a row block that has it.  Prints the number of
// sizes checked.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "../../paper_2507_06938_amd/csrc/gemv_index.hpp"

using namespace dl;

static bool row_block(int K, int kend, int klo, std::vector<int>& used) {
  constexpr int UN = 8, WAVES = 4;
  const int len = gemv_slice_len(K);
  const int sl0 = klo / len, nsl = (kend + len - 1) / len - sl0;
  if (nsl > GEMV_KS) return false;
  std::fill(used.begin(), used.end(), 0);
  for (int sl = sl0; sl < sl0 + nsl; ++sl) {
    const int k0 = sl * len, n = std::min(kend, k0 + len) - k0;
    const int kb0 = std::max(klo - k0, 0) / GEMV_STAGE * GEMV_STAGE;
    for (int kb = kb0; kb < n; kb += GEMV_STAGE) {
      const int nb = std::min(GEMV_STAGE, n - kb);
      for (int wave = 0; wave < WAVES; ++wave) {
        bool ok = true;
        auto load = [&](int k) {
          for (int u = 0; u < UN; ++u) {
            const int c = k0 + kb + gemv_column(k + 4 * u + wave, nb);
            ok = ok && c >= 0 && c < K;
          }
        };
        auto use = [&](int k) {
          for (int u = 0; u < UN; ++u)
            if (k + 4 * u + wave < nb) ++used[k0 + kb + k + 4 * u + wave];
        };
        load(0);
        load(4 * UN);
        for (int k = 0; k < nb; k += 8 * UN) {
          use(k);
          if (k + 8 * UN < nb) load(k + 8 * UN);
          use(k + 4 * UN);
          if (k + 12 * UN < nb) load(k + 12 * UN);
        }
        if (!ok) {
          std::printf("K %d kend %d klo %d slice %d: a load past the last column\n", K, kend,
                      klo, sl);
          return false;
        }
      }
    }
  }
  for (int k = 0; k < K; ++k) {
    const bool in = k >= klo && k < kend;
    if (used[k] > 1 || (in && used[k] != 1) || (k >= kend && used[k] != 0)) return false;
  }
  return true;
}

int main() {
  int sizes = 0;
  for (int K = 64; K <= 10240; K += 64) {
    std::vector<int> used(K);
    if (!row_block(K, K, 0, used)) return 1;                       // dense
    for (int RB : {128, 256})                                      // FP64, FP32 rows
      for (int r0 = 0; r0 < K; r0 += RB) {
        if (!row_block(K, std::min(K, r0 + RB), 0, used)) return 1;  // triangular
        if (!row_block(K, K, std::max(r0 - 90, 0), used)) return 1;  // begins at a band
      }
    ++sizes;
  }
  std::printf("ok %d sizes\n", sizes);
  return 0;
}
