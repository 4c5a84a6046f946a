// Dense FP64 building blocks exposed through the C ABI for testing: they run
// the same kernels as the BTA path on caller-provided matrices.  Each call
// copies its few descriptors to the device and synchronises the stream.
#include <optional>
#include <utility>
#include <vector>

#include "engine.hpp"

using namespace dl;

static GemmTask mk_task(const double* A, int64_t lda, const double* B, int64_t ldb,
                        double* C, int64_t ldc, int M, int N, int K, int flags,
                        double alpha, double beta) {
  GemmTask t{};
  t.A = A; t.B = B; t.C = C;
  t.lda = lda; t.ldb = ldb; t.ldc = ldc;
  t.M = M; t.N = N; t.K = K; t.flags = flags;
  t.alpha = alpha; t.beta = beta;
  return t;
}

template <typename T>
static hipError_t to_dev(std::vector<void*>& tmp, const std::vector<T>& h, T** d,
                         hipStream_t s) {
  if (h.empty()) return hipSuccess;
  void* p = nullptr;
  if (dev_alloc(tmp, sizeof(T) * h.size(), &p) != DL_OK) return hipErrorOutOfMemory;
  *d = (T*)p;
  return hipMemcpyAsync(p, h.data(), sizeof(T) * h.size(), hipMemcpyHostToDevice, s);
}

extern "C" dl_status dl_dgemm(int32_t transa, int32_t transb, int32_t lower,
                              int64_t M, int64_t Nn, int64_t K, double alpha,
                              const double* A, int64_t lda, const double* B,
                              int64_t ldb, double beta, double* C, int64_t ldc,
                              void* stream) {
  if (M < 0 || Nn < 0 || K < 0 || !C || (K > 0 && (!A || !B))) return DL_EINVAL;
  if (lower && M != Nn) return DL_EINVAL;
  if (M > INT32_MAX || Nn > INT32_MAX || K > INT32_MAX) return DL_EINVAL;
  if (ldc < M || (!transa && lda < M) || (transa && lda < K) ||
      (!transb && ldb < K) || (transb && ldb < Nn))
    return DL_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  int flags = (transa ? F_TA : 0) | (transb ? F_TB : 0) | (lower ? F_LOWER : 0);
  if (beta == 0.0) flags |= F_BETA0;
  std::vector<GemmTask> t{mk_task(A, lda, B, ldb, C, ldc, (int)M, (int)Nn, (int)K,
                                  flags, alpha, beta)};
  const int total = finalize_tasks(t.data(), 1);
  if (total == 0) return DL_OK;
  std::vector<void*> tmp;
  GemmTask* d = nullptr;
  hipError_t e = to_dev(tmp, t, &d, s);
  if (e == hipSuccess) e = launch_gemm_tasks(d, 1, total, s, 64, nullptr, true);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  free_all(tmp);
  return e == hipSuccess ? DL_OK : DL_EHIP;
}

// Completes the inverse of a lower-triangular factor whose diagonal tiles hold theirs,
// by recursive halving: G21 = -G22 (L21 G11), all nodes of one depth in one launch,
// deepest first.  temp: n x (nbk / 2 + 1) 64.
struct Halving {
  std::vector<GemmTask> tasks;
  std::vector<int> begin, units;  // per launch
  void add(std::vector<GemmTask> t) {
    begin.push_back((int)tasks.size());
    units.push_back(finalize_tasks(t.data(), (int)t.size()));
    tasks.insert(tasks.end(), t.begin(), t.end());
  }
  int count(size_t l) const {
    return (l + 1 < begin.size() ? begin[l + 1] : (int)tasks.size()) - begin[l];
  }
  Halving(double* A, int64_t lda, int64_t n, double* temp) {
    std::vector<std::vector<std::pair<int, int>>> levels{{{0, (int)(n / 64)}}};
    for (size_t d = 0; d < levels.size(); ++d) {
      std::vector<std::pair<int, int>> next;
      for (auto [lo, hi] : levels[d]) {
        const int mid = lo + (hi - lo) / 2;
        if (mid - lo > 1) next.push_back({lo, mid});
        if (hi - mid > 1) next.push_back({mid, hi});
      }
      if (!next.empty()) levels.push_back(next);
    }
    for (size_t d = levels.size(); d-- > 0;) {
      std::vector<GemmTask> tT, tG;
      for (auto [lo, hi] : levels[d]) {
        const int mid = lo + (hi - lo) / 2, n1 = (mid - lo) * 64, n2 = (hi - mid) * 64;
        double* L21 = A + (int64_t)mid * 64 + (int64_t)lo * 64 * lda;
        double* G11 = A + (int64_t)lo * 64 * (lda + 1);
        double* G22 = A + (int64_t)mid * 64 * (lda + 1);
        double* T = temp + (int64_t)lo * 64;
        tT.push_back(mk_task(L21, lda, G11, lda, T, n, n2, n1, n1, F_KLO_COL | F_BETA0, 1.0, 0.0));
        tG.push_back(mk_task(G22, lda, T, n, L21, lda, n2, n1, n2, F_KHI_ROW | F_BETA0, -1.0, 0.0));
      }
      add(tT);
      add(tG);
    }
  }
};

// Most tiles of a block whose inverse dl_dpotrf forms beside the factor.  That reads
// and writes every accumulator once per panel, n^3 / 6 / 64^3 tiles three times over,
// which beyond takes longer than a few launches of large products after the factor
// (beside / after in ms: n = 3072 1.37 / 1.62, 4096 2.49 / 2.72, 4608 3.49 / 3.40, 6144
// 7.06 / 6.05, 8192 17.4 / 12.7).
constexpr int kBesideTiles = 64;

// Right-looking blocked Cholesky, a launch per panel of 64 columns (PanelTask),
// with want_inverse the inverse beside it, or of large blocks after it.  One block is
// bound by the chain of its tile factors (20 us a panel): 32 tiles take 0.71 ms, where a
// launch each for the factor, the solve and the update of every panel and the inverse
// by recursive halving after it took 1.25.
extern "C" dl_status dl_dpotrf(int64_t n, double* A, int64_t lda,
                               int32_t want_inverse, double* logdet_dev,
                               int64_t* info_dev, void* stream) {
  if (n <= 0 || n % 64 != 0 || n > (1 << 20) || !A || lda < n || !logdet_dev ||
      !info_dev)
    return DL_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  const int nbk = (int)(n / 64);
  std::vector<void*> tmp;
  double *Gd = nullptr, *temp = nullptr, *logdiag = nullptr, *part = nullptr;
  const bool inv = want_inverse != 0, after = inv && nbk > kBesideTiles;
  const size_t acc = !inv ? 0 : (after ? (size_t)nbk * (nbk / 2 + 1) : (size_t)nbk * (nbk - 1) / 2);
  if (dev_alloc(tmp, sizeof(double) * 4096, (void**)&Gd) != DL_OK ||
      dev_alloc(tmp, sizeof(double) * 4096 * (2 + acc), (void**)&temp) != DL_OK ||
      dev_alloc(tmp, sizeof(double) * n, (void**)&logdiag) != DL_OK ||
      dev_alloc(tmp, sizeof(double) * SUM_BLOCKS, (void**)&part) != DL_OK) {
    free_all(tmp);
    return DL_ENOMEM;
  }
  std::vector<MiscJob> pre(2);
  pre[0].kind = MJ_ZERO_I64; pre[0].dst = (double*)info_dev; pre[0].n = 1;
  pre[1].kind = MJ_ZERO_UPPER_TILES; pre[1].dst = A; pre[1].rows = (int)n; pre[1].ldd = lda;
  // tile 0 (mode 0: A <- L, its inverse to Gd; mode 1: inverse in place) and the
  // panel below it, then the panel steps
  std::vector<PotrfTileArgs> pt(1);
  PotrfTileArgs& a = pt[0];
  a.A = A;
  a.lda = lda;
  a.Ginv = inv ? nullptr : Gd;
  a.logdiag = logdiag;
  a.info = info_dev;
  a.row0 = 0;
  a.mode = inv ? 1 : 0;
  std::vector<GemmTask> solve;
  std::vector<PanelTask> steps(nbk > 1 ? nbk : 0);
  std::vector<int> grid(nbk);
  int units = 0, nsteps = 0;
  std::vector<MiscJob> post;
  if (nbk > 1) {
    solve.push_back(mk_task(A + 64, lda, inv ? A : Gd, inv ? lda : 64, A + 64, lda, (int)n - 64,
                            64, 64, F_TB | F_BETA0, 1.0, 0.0));
    units = finalize_tasks(solve.data(), 1);
    nsteps = panel_steps(n, A, lda, after ? PANEL_DIAG : (inv ? PANEL_INVERSE : PANEL_L), logdiag,
                         info_dev, temp, steps.data(), grid.data());
    if (inv && !after) post.push_back(last_inverse_tile(n, A, lda, temp));
  }
  std::optional<Halving> halves;
  if (after) halves.emplace(A, lda, n, temp);
  std::vector<SumJob> sj(1);
  sj[0].src = logdiag; sj[0].n = n; sj[0].scale = 2.0; sj[0].dst = logdet_dev; sj[0].partial = part;
  MiscJob *dpre = nullptr, *dpost = nullptr;
  PotrfTileArgs* dpt = nullptr;
  GemmTask* dt = nullptr;
  PanelTask* dst = nullptr;
  GemmTask* dh = nullptr;
  SumJob* dsj = nullptr;
  hipError_t e = to_dev(tmp, pre, &dpre, s);
  if (e == hipSuccess) e = to_dev(tmp, pt, &dpt, s);
  if (e == hipSuccess) e = to_dev(tmp, solve, &dt, s);
  if (e == hipSuccess) e = to_dev(tmp, steps, &dst, s);
  if (e == hipSuccess) e = to_dev(tmp, post, &dpost, s);
  if (e == hipSuccess && after) e = to_dev(tmp, halves->tasks, &dh, s);
  if (e == hipSuccess) e = to_dev(tmp, sj, &dsj, s);
  if (e == hipSuccess) e = launch_misc(dpre, 2, s);
  if (e == hipSuccess) e = launch_potrf_tiles(dpt, 1, s);
  if (e == hipSuccess) e = launch_gemm_tasks(dt, (int)solve.size(), units, s);
  for (int j = 0; j < nsteps && e == hipSuccess; ++j)
    e = launch_panel_step(dst + j, grid[j], s);
  if (e == hipSuccess && !post.empty()) e = launch_misc(dpost, 1, s);
  for (size_t l = 0; after && l < halves->begin.size() && e == hipSuccess; ++l)
    e = launch_gemm_tasks(dh + halves->begin[l], halves->count(l), halves->units[l], s);
  if (e == hipSuccess) e = launch_sums(dsj, 1, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  free_all(tmp);
  return e == hipSuccess ? DL_OK : DL_EHIP;
}
