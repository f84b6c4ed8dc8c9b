// Phasing (section II-D): the density rho on an N^3 grid and its Fourier
// coefficients are driven back and forth between the real-space constraints
// (support, positivity) and the measured amplitudes, by error reduction (ER)
// and hybrid input-output (HIO) steps, with shrinkwrap support updates.
// The 3D transforms are three separable line transforms each (numpy's
// convention: forward e^{-2 pi i k.r / N}, inverse with 1 / N per axis) on the
// nonnegative half of the Hermitian spectrum along axis 2; the amplitude
// projection runs between the two axis-0 transforms of an iteration, in one
// pass with them, and the real-space step in the last pass of the inverse
// transform.  The shrinkwrap blur is three separable circular convolutions with
// the periodic Gaussian, as contractions with its circulant table.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <new>
#include <set>
#include <string>
#include <vector>

#include "dft.h"
#include "internal.h"

namespace spfel {

constexpr int kPhBlocks = 256;

struct Phase {
  int device = 0, N = 0;
  DftTable fwd;           // exp(-2 pi i k l / N)
  DftTable inv;           // exp(+2 pi i k l / N) / N
  float2 *Wg = nullptr;   // [N][N] circulant Gaussian g[(k - l) mod N]
  float2 *T1 = nullptr, *T2 = nullptr;   // N^3 each: transform intermediates
  float2 *F = nullptr;    // [N][N][N / 2 + 1]: the spectrum, where the fused axis-0 pass does not fit
  float *rp = nullptr;    // N^3: |rho| of the blur
  float *bl = nullptr;    // N^3: the blurred |rho|
  float *part = nullptr;  // partial sums of the error (or of the blur's maximum)
  size_t bytes = 0;
};

static std::mutex g_pmu;
static std::set<Phase *> g_plive;

static bool plive(Phase *p) {
  std::lock_guard<std::mutex> lk(g_pmu);
  return p && g_plive.count(p) > 0;
}

static void free_phase(Phase *p) {
  void *bufs[] = {p->fwd.t, p->inv.t, p->Wg, p->F, p->T1, p->T2, p->rp, p->bl, p->part};
  for (void *b : bufs)
    if (b) (void)hipFree(b);
}

// ---------------------------------------------------------------- kernels --

// |rho| (the blur's first contraction reads float input).
__global__ __launch_bounds__(256) void abs_kernel(const float *__restrict__ rho, int64_t n,
                                                  float *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = fabsf(rho[i]);
}

// Circulant table of the periodic Gaussian: W[l][k] = g[(k - l) mod N],
// g[d] ~ exp(-d^2 / (2 sigma^2)) with d the signed periodic offset, unit sum
// (float64, rounded once).  One block.
__global__ __launch_bounds__(256) void gaussian_table_kernel(int N, double sigma,
                                                             float2 *__restrict__ W) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int j = threadIdx.x; j < N; j += 256) {
    const double d = j <= N / 2 ? j : j - N;
    s += exp(-d * d / (2.0 * sigma * sigma));
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
    __syncthreads();
  }
  const double total = sh[0];
  for (int64_t t = threadIdx.x; t < (int64_t)N * N; t += 256) {
    const int l = (int)(t / N), k = (int)(t - (int64_t)l * N);
    int j = k - l;
    j += j < 0 ? N : 0;
    const double d = j <= N / 2 ? j : j - N;
    W[t] = make_float2((float)(exp(-d * d / (2.0 * sigma * sigma)) / total), 0.f);
  }
}

// Partial maxima of b (fixed order), then support = b >= tau max.
__global__ __launch_bounds__(256) void max_partial_kernel(const float *__restrict__ b, int64_t n,
                                                          float *__restrict__ part) {
  __shared__ float sh[256];
  const int64_t per = (n + kPhBlocks - 1) / kPhBlocks;
  const int64_t lo = (int64_t)blockIdx.x * per, hi = min(n, lo + per);
  float m = 0.f;   // b >= 0
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256) m = fmaxf(m, b[i]);
  sh[threadIdx.x] = m;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) sh[threadIdx.x] = fmaxf(sh[threadIdx.x], sh[threadIdx.x + st]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(256) void threshold_kernel(const float *__restrict__ b, int64_t n,
                                                        const float *__restrict__ part, float tau,
                                                        uint8_t *__restrict__ support) {
  __shared__ float thr;
  if (threadIdx.x == 0) {
    float m = 0.f;
    for (int j = 0; j < kPhBlocks; ++j) m = fmaxf(m, part[j]);
    thr = tau * m;
  }
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) support[i] = b[i] >= thr ? 1 : 0;
}

static dim3 pgrid(int64_t n) { return dim3((unsigned)((n + 255) / 256)); }

// One iteration: rho to the half spectrum (axes 2, 1), the axis-0 pass with
// the projection, back (axes 1, 2) and the real-space step.
static hipError_t iteration(const Phase &p, float *rho, const float *amp, const uint8_t *measured,
                            const uint8_t *support, int hio, float beta, int positivity, float *err,
                            hipStream_t st) {
  const int N = p.N, half = N / 2 + 1;
  const int64_t cols = (int64_t)N * half;
  const DftLines lines{(int64_t)N * N, 1, N, half}, back{(int64_t)N * N, 1, half, N};
  const DftLines axis1{cols, half, N, N}, axis0{cols, (int)cols, N, N};
  DftEpilogue none, last, reduce;
  hipError_t e = launch_dft(p.fwd, kRH, lines, rho, p.T1, none, st);
  if (e == hipSuccess) e = launch_dft(p.fwd, kCC, axis1, p.T1, p.T2, none, st);
  if (e != hipSuccess) return e;
  if (!p.F) {
    e = launch_dft_phase(p.fwd, p.inv, p.T2, amp, measured, p.part, st);
  } else {
    e = launch_dft(p.fwd, kCC, axis0, p.T2, p.F, none, st);
    if (e == hipSuccess) e = launch_phase_projection(N, p.F, amp, measured, p.part, st);
    if (e == hipSuccess) e = launch_dft(p.inv, kCC, axis0, p.F, p.T2, none, st);
  }
  if (e != hipSuccess) return e;
  reduce.err_part = p.part;
  reduce.err_n = (int)dft_phase_parts(N);
  reduce.err = err;
  e = launch_dft(p.inv, kCC, axis1, p.T2, p.T1, reduce, st);
  if (e != hipSuccess) return e;
  last.support = support;
  last.hio = hio;
  last.beta = beta;
  last.positivity = positivity;
  return launch_dft(p.inv, kHR, back, p.T1, rho, last, st);
}

}  // namespace spfel

using namespace spfel;

extern "C" {

int spfel_phase_create(spfel_phase *out, int n, int device) {
  clear_error();
  if (!out) return fail(SPFEL_EINVAL, "phase_create: out is NULL");
  *out = nullptr;
  if (n < 2) return fail(SPFEL_EINVAL, "phase_create: n must be >= 2");
  if (n > 1024) return fail(SPFEL_ERANGE, "phase_create: n > 1024");
  int ndev = 0;
  hipError_t e = hipGetDeviceCount(&ndev);
  if (e != hipSuccess) return hip_fail(e, "phase_create: hipGetDeviceCount");
  if (device < 0 || device >= ndev) return fail(SPFEL_EINVAL, "phase_create: no such device");
  int prev = 0;
  (void)hipGetDevice(&prev);
  if (prev != device) (void)hipSetDevice(device);
  Phase *p = new (std::nothrow) Phase();
  if (!p) return fail(SPFEL_ENOMEM, "phase_create: host allocation");
  p->device = device;
  p->N = n;
  const size_t N = n, N3 = N * N * N;
  const size_t tab = dft_table_sizes(p->fwd, kCyclic, 0, n);
  (void)dft_table_sizes(p->inv, kCyclic, 0, n);
  const size_t parts = 2 * std::max<size_t>((size_t)dft_phase_parts(n), kPhBlocks);
  struct Req {
    void **ptr;
    size_t bytes;
  } reqs[] = {{reinterpret_cast<void **>(&p->fwd.t), tab},
              {reinterpret_cast<void **>(&p->inv.t), tab},
              {reinterpret_cast<void **>(&p->Wg), N * N * 8},
              {reinterpret_cast<void **>(&p->T1), N3 * 8},
              {reinterpret_cast<void **>(&p->T2), N3 * 8},
              {reinterpret_cast<void **>(&p->F), dft_phase_fits(p->fwd) ? 0 : N * N * (N / 2 + 1) * 8},
              {reinterpret_cast<void **>(&p->rp), N3 * 4},
              {reinterpret_cast<void **>(&p->bl), N3 * 4},
              {reinterpret_cast<void **>(&p->part), parts * 4}};
  for (auto &r : reqs) {
    if (r.bytes == 0) continue;
    e = hipMalloc(r.ptr, r.bytes);
    if (e != hipSuccess) {
      *r.ptr = nullptr;
      (void)hipGetLastError();
      free_phase(p);
      delete p;
      if (prev != device) (void)hipSetDevice(prev);
      return fail(SPFEL_ENOMEM, std::string("phase_create: hipMalloc: ") + hipGetErrorString(e));
    }
    p->bytes += r.bytes;
  }
  const double scale = 1.0 / (double)n;
  e = dft_table_fill(p->fwd, -1, false, [](int) { return 1.0; });
  if (e == hipSuccess) e = dft_table_fill(p->inv, +1, false, [&](int) { return scale; });
  if (prev != device) (void)hipSetDevice(prev);
  if (e != hipSuccess) {
    free_phase(p);
    delete p;
    return hip_fail(e, "phase_create: table upload");
  }
  {
    std::lock_guard<std::mutex> lk(g_pmu);
    g_plive.insert(p);
  }
  *out = reinterpret_cast<spfel_phase>(p);
  return SPFEL_OK;
}

int spfel_phase_destroy(spfel_phase h) {
  clear_error();
  Phase *p = reinterpret_cast<Phase *>(h);
  {
    std::lock_guard<std::mutex> lk(g_pmu);
    if (!p || g_plive.erase(p) == 0) return fail(SPFEL_ESTATE, "phase_destroy: not a live object");
  }
  free_phase(p);
  delete p;
  return SPFEL_OK;
}

int spfel_phase_iterate(spfel_phase h, float *rho, const float *amp, const uint8_t *measured,
                        const uint8_t *support, int n_iter, int mode, float beta,
                        int positivity, float *err, void *stream) {
  clear_error();
  Phase *p = reinterpret_cast<Phase *>(h);
  if (!plive(p)) return fail(SPFEL_ESTATE, "phase_iterate: not a live object");
  if (!rho || !amp || !support) return fail(SPFEL_EINVAL, "phase_iterate: NULL pointer");
  if (mode != SPFEL_PHASE_ER && mode != SPFEL_PHASE_HIO)
    return fail(SPFEL_EINVAL, "phase_iterate: mode must be ER or HIO");
  if (n_iter < 0) return fail(SPFEL_EINVAL, "phase_iterate: negative n_iter");
  if (!std::isfinite(beta)) return fail(SPFEL_EINVAL, "phase_iterate: beta not finite");
  if ((reinterpret_cast<uintptr_t>(rho) & 3) || (reinterpret_cast<uintptr_t>(amp) & 3) ||
      (err && (reinterpret_cast<uintptr_t>(err) & 3)))
    return fail(SPFEL_EINVAL, "phase_iterate: misaligned float array");
  hipStream_t st = static_cast<hipStream_t>(stream);
  for (int it = 0; it < n_iter; ++it) {
    hipError_t e = iteration(*p, rho, amp, measured, support, mode == SPFEL_PHASE_HIO ? 1 : 0, beta,
                             positivity ? 1 : 0, err ? err + it : nullptr, st);
    if (e != hipSuccess) return hip_fail(e, "phase_iterate: launch");
  }
  return SPFEL_OK;
}

int spfel_phase_shrinkwrap(spfel_phase h, const float *rho, float sigma, float tau,
                           uint8_t *support, float *blurred, void *stream) {
  clear_error();
  Phase *p = reinterpret_cast<Phase *>(h);
  if (!plive(p)) return fail(SPFEL_ESTATE, "phase_shrinkwrap: not a live object");
  if (!rho || !support) return fail(SPFEL_EINVAL, "phase_shrinkwrap: NULL pointer");
  if (!(sigma > 0.f) || !std::isfinite(sigma)) return fail(SPFEL_EINVAL, "phase_shrinkwrap: sigma must be > 0");
  if (!(tau >= 0.f && tau <= 1.f)) return fail(SPFEL_EINVAL, "phase_shrinkwrap: tau must be in [0, 1]");
  if ((reinterpret_cast<uintptr_t>(rho) & 3) || (blurred && (reinterpret_cast<uintptr_t>(blurred) & 3)))
    return fail(SPFEL_EINVAL, "phase_shrinkwrap: misaligned float array");
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int N = p->N;
  const int64_t n3 = (int64_t)N * N * N;
  float *b = blurred ? blurred : p->bl;
  hipLaunchKernelGGL(gaussian_table_kernel, dim3(1), dim3(256), 0, st, N, (double)sigma, p->Wg);
  float *absr = p->rp;
  hipLaunchKernelGGL(abs_kernel, pgrid(n3), dim3(256), 0, st, rho, n3, absr);
  hipError_t e = launch_contract(absr, false, p->Wg, p->T1, 0, N * N, N, N, 1, st);
  if (e == hipSuccess) e = launch_contract(p->T1, true, p->Wg, p->T2, 0, N, N, N, N, st);
  if (e == hipSuccess) e = launch_contract(p->T2, true, p->Wg, b, 1, 1, N, N, N * N, st);
  if (e != hipSuccess) return hip_fail(e, "phase_shrinkwrap: launch");
  hipLaunchKernelGGL(max_partial_kernel, dim3(kPhBlocks), dim3(256), 0, st, b, n3, p->part);
  hipLaunchKernelGGL(threshold_kernel, pgrid(n3), dim3(256), 0, st, b, n3, p->part, tau, support);
  e = hipGetLastError();
  return e == hipSuccess ? SPFEL_OK : hip_fail(e, "phase_shrinkwrap: launch");
}

}  // extern "C"
