// dl_dpotrf_noalloc: the dense Cholesky of dl_dpotrf for callers that cannot
// allocate device memory.  Its temporaries (the panel steps' side ring, the
// inverse's accumulators, the first tile's inverse, the log-diagonal, the
// reduction partials and the launch descriptors) live in one file-scope
// device array instead of per-call allocations; the kernels are the same as
// dl_dpotrf's and receive the array's device address like any other buffer.
#include <string.h>

#include <mutex>

#include "engine.hpp"

using namespace dl;

namespace {

constexpr int64_t kMaxN = DL_DPOTRF_NOALLOC_MAX_N;
constexpr int kMaxTiles = (int)(kMaxN / 64);
// the descriptors of one call, each rounded up to 256 bytes
constexpr size_t kDescBytes = 256 * 6 + sizeof(PanelTask) * kMaxTiles + 256;
// scratch layout, in doubles (every region 256-byte aligned)
constexpr int64_t kDescDoubles = 8192;  // 64 KiB of launch descriptors
constexpr int64_t kGdDoubles = 4096;
constexpr int64_t kTempDoubles = 4096 * (2 + (int64_t)kMaxTiles * (kMaxTiles - 1) / 2);
constexpr int64_t kLogDoubles = kMaxN;
constexpr int64_t kPartDoubles = 256;
constexpr int64_t kScratchDoubles =
    kDescDoubles + kGdDoubles + kTempDoubles + kLogDoubles + kPartDoubles;
static_assert(kDescBytes <= kDescDoubles * 8 && sizeof(MiscJob) <= 256 &&
                  sizeof(GemmTask) <= 256 && sizeof(SumJob) <= 256,
              "descriptors");
static_assert(kScratchDoubles * 8 == DL_DPOTRF_NOALLOC_SCRATCH_BYTES,
              "scratch size stated in the header");

}  // namespace

// The scratch array.  In host code this name is only a stand-in for the
// symbol: its device address comes from hipGetSymbolAddress (one per device).
static __device__ __align__(256) double scratch[kScratchDoubles];

namespace {

std::mutex g_mu;
double* g_scratch[64] = {nullptr};

// Device address of `scratch` on the current device (looked up once).
dl_status scratch_ptr(double** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return DL_EHIP;
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return DL_EHIP;
    g_scratch[dev] = (double*)p;
  }
  *out = g_scratch[dev];
  return DL_OK;
}

// Host -> device copy of a few KB through kernel arguments (captured by value
// at launch), so the host array may go away when the launch call returns.
constexpr int kChunkWords = 768;
struct Chunk {
  uint32_t w[kChunkWords];
};

__global__ __launch_bounds__(256) void k_put_words(uint32_t* __restrict__ dst, Chunk c,
                                                   int nwords) {
  for (int i = threadIdx.x; i < nwords; i += 256) dst[i] = c.w[i];
}

hipError_t put_bytes(void* dst, const void* src, size_t bytes, hipStream_t s) {
  const uint32_t* w = (const uint32_t*)src;
  size_t words = (bytes + 3) / 4;
  uint32_t* d = (uint32_t*)dst;
  while (words > 0) {
    const int nw = (int)(words < (size_t)kChunkWords ? words : (size_t)kChunkWords);
    Chunk c;
    for (int i = 0; i < nw; ++i) c.w[i] = w[i];
    hipLaunchKernelGGL(k_put_words, dim3(1), dim3(256), 0, s, d, c, nw);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    w += nw;
    d += nw;
    words -= nw;
  }
  return hipSuccess;
}

// One buffer for the call's descriptors on both sides: put() appends host
// values and returns the device address they will have.
struct DescBuffer {
  alignas(256) char host[kDescBytes];
  char* dev;
  size_t used = 0;
  template <typename T>
  T* put(const T* v, int count) {
    T* p = (T*)(dev + used);
    memcpy(host + used, v, sizeof(T) * (size_t)count);
    used += ((sizeof(T) * (size_t)count + 255) / 256) * 256;
    return p;
  }
};

GemmTask task(const double* A, int64_t lda, const double* B, int64_t ldb, double* C,
              int64_t ldc, int M, int N, int K, int flags, double alpha, double beta) {
  GemmTask t{};
  t.A = A; t.B = B; t.C = C;
  t.lda = lda; t.ldb = ldb; t.ldc = ldc;
  t.M = M; t.N = N; t.K = K; t.flags = flags;
  t.alpha = alpha; t.beta = beta;
  return t;
}

}  // namespace

extern "C" dl_status dl_dpotrf_noalloc(int64_t n, double* A, int64_t lda,
                                       int32_t want_inverse, double* logdet_dev,
                                       int64_t* info_dev, void* stream) {
  if (n <= 0 || n % 64 != 0 || n > kMaxN || !A || lda < n || !logdet_dev || !info_dev)
    return DL_EINVAL;
  double* ptr = nullptr;
  const dl_status st = scratch_ptr(&ptr);
  if (st != DL_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  const int nbk = (int)(n / 64);

  // regions of the scratch array (device addresses)
  double* Gd = ptr + kDescDoubles;
  double* temp = Gd + kGdDoubles;
  double* logdiag = temp + kTempDoubles;
  double* part = logdiag + kLogDoubles;

  // host descriptors, in fixed-size arrays
  MiscJob pre[2] = {};
  pre[0].kind = MJ_ZERO_I64; pre[0].dst = (double*)info_dev; pre[0].n = 1;
  pre[1].kind = MJ_ZERO_UPPER_TILES; pre[1].dst = A; pre[1].rows = (int)n; pre[1].ldd = lda;
  // as dl_dpotrf: tile 0 (mode 0: A <- L, its inverse to Gd; mode 1: inverse in
  // place), the panel below it, the panel steps
  const bool inv = want_inverse != 0;
  PotrfTileArgs pt{};
  pt.A = A;
  pt.lda = lda;
  pt.Ginv = inv ? nullptr : Gd;
  pt.logdiag = logdiag;
  pt.info = info_dev;
  pt.mode = inv ? 1 : 0;
  GemmTask solve{};
  PanelTask steps[kMaxTiles];
  int grid[kMaxTiles], units = 0, nsteps = 0;
  MiscJob post{};
  if (nbk > 1) {
    solve = task(A + 64, lda, inv ? A : Gd, inv ? lda : 64, A + 64, lda, (int)n - 64, 64, 64,
                 F_TB | F_BETA0, 1.0, 0.0);
    units = finalize_tasks(&solve, 1);
    nsteps = panel_steps(n, A, lda, inv ? PANEL_INVERSE : PANEL_L, logdiag, info_dev, temp, steps, grid);
    if (inv) post = last_inverse_tile(n, A, lda, temp);
  }
  SumJob sj{};
  sj.src = logdiag; sj.n = n; sj.scale = 2.0; sj.dst = logdet_dev; sj.partial = part;

  // descriptors into the scratch array, then the launches of dl_dpotrf
  DescBuffer buf;
  buf.dev = (char*)ptr;
  MiscJob* dpre = buf.put(pre, 2);
  PotrfTileArgs* dpt = buf.put(&pt, 1);
  GemmTask* dt = buf.put(&solve, 1);
  PanelTask* dst = buf.put(steps, nsteps);
  MiscJob* dpost = buf.put(&post, 1);
  SumJob* dsj = buf.put(&sj, 1);
  hipError_t e = put_bytes(ptr, buf.host, buf.used, s);
  if (e == hipSuccess) e = launch_misc(dpre, 2, s);
  if (e == hipSuccess) e = launch_potrf_tiles(dpt, 1, s);
  if (e == hipSuccess && nbk > 1) e = launch_gemm_tasks(dt, 1, units, s);
  for (int j = 0; j < nsteps && e == hipSuccess; ++j)
    e = launch_panel_step(dst + j, grid[j], s);
  if (e == hipSuccess && nbk > 1 && inv) e = launch_misc(dpost, 1, s);
  if (e == hipSuccess) e = launch_sums(dsj, 1, s);
  return e == hipSuccess ? DL_OK : DL_EHIP;
}
