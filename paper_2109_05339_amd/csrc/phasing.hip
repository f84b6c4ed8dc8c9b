// Phasing (section II-D): the density rho on an N^3 grid and its Fourier
// coefficients are driven back and forth between the real-space constraints
// (support, positivity) and the measured amplitudes, by error reduction (ER)
// and hybrid input-output (HIO) steps, with shrinkwrap support updates.
// The 3D transforms are separable (numpy's convention: forward
// e^{-2 pi i k.r / N}, inverse with 1 / N per axis).  Error reduction runs on
// folded line transforms and the nonnegative half of the Hermitian spectrum
// along axis 2: the amplitude projection lies between the two axis-0
// transforms of an iteration, in one pass with them, and the real-space step in
// the last pass of the inverse transform.  HIO and the shrinkwrap blur (three
// circular convolutions with the periodic Gaussian) are contractions with full
// tables.
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
  DftTable inv;           // exp(+2 pi i k l / N) / N, behind fwd
  bool fused = false;     // whether the axis-0 pass of error reduction fits the LDS
  float2 *Wf = nullptr;   // [N][N] exp(-2 pi i k l / N)
  float2 *Wi = nullptr;   // [N][N] exp(+2 pi i k l / N) / N, behind Wf
  float2 *Wg = nullptr;   // [N][N] circulant Gaussian g[(k - l) mod N]
  float2 *F = nullptr, *T1 = nullptr, *T2 = nullptr;   // N^3 each
  float *rp = nullptr;    // N^3: rho' (or the blurred |rho|)
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
  void *bufs[] = {p->fwd.t, p->Wf, p->Wg, p->F, p->T1, p->T2, p->rp, p->part};
  for (void *b : bufs)
    if (b) (void)hipFree(b);
}

// ---------------------------------------------------------------- kernels --

// Reciprocal-space projection, in place on F: where measured, F <- A F / |F|
// (A where F = 0); elsewhere F is kept.  Partial sums of (|F| - A)^2 and A^2
// over measured coefficients, fixed order (block b takes a contiguous range,
// 256 strided partials, a pairwise tree).
__global__ __launch_bounds__(256) void amplitude_projection_kernel(
    float2 *__restrict__ F, const float *__restrict__ amp, const uint8_t *__restrict__ measured,
    int64_t n, float *__restrict__ part) {
  __shared__ float sh[2][256];
  const int64_t per = (n + kPhBlocks - 1) / kPhBlocks;
  const int64_t lo = (int64_t)blockIdx.x * per, hi = min(n, lo + per);
  float e = 0.f, a2 = 0.f;
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
    if (measured && !measured[i]) continue;
    const float2 f = F[i];
    const float A = amp[i];
    const float mag = sqrtf(fmaf(f.x, f.x, f.y * f.y));
    const float d = mag - A;
    e = fmaf(d, d, e);
    a2 = fmaf(A, A, a2);
    F[i] = mag > 0.f ? make_float2(A * (f.x / mag), A * (f.y / mag)) : make_float2(A, 0.f);
  }
  sh[0][threadIdx.x] = e;
  sh[1][threadIdx.x] = a2;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      sh[0][threadIdx.x] += sh[0][threadIdx.x + st];
      sh[1][threadIdx.x] += sh[1][threadIdx.x + st];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[blockIdx.x] = sh[0][0];
    part[kPhBlocks + blockIdx.x] = sh[1][0];
  }
}

// *err = (sum of the error partials) / (sum of the A^2 partials).
__global__ void phase_error_kernel(const float *__restrict__ part, float *__restrict__ err) {
  if (threadIdx.x != 0) return;
  float e = 0.f, a = 0.f;
  for (int b = 0; b < kPhBlocks; ++b) {
    e += part[b];
    a += part[kPhBlocks + b];
  }
  *err = a > 0.f ? e / a : 0.f;
}

// Real-space step of HIO: where the constraint holds (support, and rho' >= 0
// with positivity) rho <- rho'; elsewhere rho <- rho - beta rho'.
__global__ __launch_bounds__(256) void hio_kernel(float *__restrict__ rho, const float *__restrict__ rp,
                                                  const uint8_t *__restrict__ support, int64_t n,
                                                  float beta, int positivity) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float v = rp[i];
  const bool holds = support[i] && (!positivity || v >= 0.f);
  rho[i] = holds ? v : fmaf(-beta, v, rho[i]);
}

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

// 3D transform of rho (real) into F.
static hipError_t forward3(const Phase &p, const float *rho, hipStream_t st) {
  const int N = p.N;
  hipError_t e = launch_contract_rows(rho, false, p.Wf, p.T1, N * N, N, N, st);
  if (e == hipSuccess) e = launch_contract(p.T1, p.Wf, p.T2, false, N, N, N, N, st);
  if (e == hipSuccess) e = launch_contract(p.T2, p.Wf, p.F, false, 1, N, N, N * N, st);
  return e;
}

// Real part of the inverse transform of F into out.
static hipError_t inverse3(const Phase &p, float *out, hipStream_t st) {
  const int N = p.N;
  hipError_t e = launch_contract_rows(p.F, true, p.Wi, p.T1, N * N, N, N, st);
  if (e == hipSuccess) e = launch_contract(p.T1, p.Wi, p.T2, false, N, N, N, N, st);
  if (e == hipSuccess) e = launch_contract(p.T2, p.Wi, out, true, 1, N, N, N * N, st);
  return e;
}

// One HIO iteration, by full tables.  Its feedback outside the support
// amplifies rounding some tenfold every two iterations: the line transforms'
// order of sums changes the density by 3e-5 to 6e-5 of itself after six
// iterations and by 1e-3 to 3e-3 after twelve (N = 129; error reduction: 2e-6
// after ten).  So the density that a sequence of HIO steps arrives at keeps its
// order of sums (330 us per iteration at N = 129, where the line transforms take
// 70), although the line transforms mostly land nearer to float64 (after twelve
// iterations 0.7e-3 to 1.3e-3 away from it instead of 1.1e-3 to 2.2e-3).
static hipError_t hio_iteration(const Phase &p, float *rho, const float *amp, const uint8_t *measured,
                                const uint8_t *support, float beta, int positivity, float *err,
                                hipStream_t st) {
  const int64_t n3 = (int64_t)p.N * p.N * p.N;
  hipError_t e = forward3(p, rho, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(amplitude_projection_kernel, dim3(kPhBlocks), dim3(256), 0, st, p.F, amp, measured,
                     n3, p.part);
  if (err) hipLaunchKernelGGL(phase_error_kernel, dim3(1), dim3(64), 0, st, p.part, err);
  e = inverse3(p, p.rp, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(hio_kernel, pgrid(n3), dim3(256), 0, st, rho, p.rp, support, n3, beta, positivity);
  return hipGetLastError();
}

// One iteration of error reduction: rho to the half spectrum (axes 2, 1), the axis-0 pass with
// the projection, back (axes 1, 2) and the real-space step.
static hipError_t er_iteration(const Phase &p, float *rho, const float *amp, const uint8_t *measured,
                               const uint8_t *support, int positivity, float *err, hipStream_t st) {
  const int N = p.N, half = N / 2 + 1;
  const int64_t cols = (int64_t)N * half;
  const DftLines lines{(int64_t)N * N, 1, N, half}, back{(int64_t)N * N, 1, half, N};
  const DftLines axis1{cols, half, N, N}, axis0{cols, (int)cols, N, N};
  DftEpilogue none, last, reduce;
  hipError_t e = launch_dft(p.fwd, kRH, lines, rho, p.T1, none, st);
  if (e == hipSuccess) e = launch_dft(p.fwd, kCC, axis1, p.T1, p.T2, none, st);
  if (e != hipSuccess) return e;
  if (p.fused) {
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
  p->fused = dft_phase_fits(p->fwd);
  const size_t parts = 2 * std::max<size_t>((size_t)dft_phase_parts(n), kPhBlocks);
  struct Req {
    void **ptr;
    size_t bytes;
  } reqs[] = {{reinterpret_cast<void **>(&p->fwd.t), 2 * tab},
              {reinterpret_cast<void **>(&p->Wf), 2 * N * N * 8},
              {reinterpret_cast<void **>(&p->Wg), N * N * 8},
              {reinterpret_cast<void **>(&p->F), N3 * 8},
              {reinterpret_cast<void **>(&p->T1), N3 * 8},
              {reinterpret_cast<void **>(&p->T2), N3 * 8},
              {reinterpret_cast<void **>(&p->rp), N3 * 4},
              {reinterpret_cast<void **>(&p->part), parts * 4}};
  for (auto &r : reqs) {
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
  const size_t nt = tab / sizeof(float2);
  p->inv.t = p->fwd.t + nt;
  p->Wi = p->Wf + N * N;
  std::vector<float2> lines(2 * nt);
  dft_table_values(p->fwd, -1, [](int) { return 1.0; }, lines.data());
  dft_table_values(p->inv, +1, [&](int) { return scale; }, lines.data() + nt);
  e = hipMemcpy(p->fwd.t, lines.data(), 2 * tab, hipMemcpyHostToDevice);
  // DFT tables in float64 with the phase index reduced modulo N exactly: N
  // distinct entries (a cosine and a sine for each of the N^2 took most of the
  // creation: 0.56 ms at N = 129, 0.10 here)
  std::vector<float2> wf(N), wi(N), W(2 * N * N);
  for (size_t j = 0; j < N; ++j) {
    const double a = 2.0 * M_PI * (double)j / (double)N;
    wf[j] = make_float2((float)std::cos(a), (float)-std::sin(a));
    wi[j] = make_float2((float)(std::cos(a) / (double)N), (float)(std::sin(a) / (double)N));
  }
  for (size_t l = 0; l < N; ++l)
    for (size_t k = 0, j = 0; k < N; ++k) {   // j = l k mod N
      W[l * N + k] = wf[j];
      W[N * N + l * N + k] = wi[j];
      j += l;
      j -= j >= N ? N : 0;
    }
  if (e == hipSuccess) e = hipMemcpy(p->Wf, W.data(), 2 * N * N * 8, hipMemcpyHostToDevice);
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
    float *const er = err ? err + it : nullptr;
    const hipError_t e = mode == SPFEL_PHASE_HIO
                             ? hio_iteration(*p, rho, amp, measured, support, beta, positivity ? 1 : 0, er, st)
                             : er_iteration(*p, rho, amp, measured, support, positivity ? 1 : 0, er, st);
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
  float *b = blurred ? blurred : p->rp;
  hipLaunchKernelGGL(gaussian_table_kernel, dim3(1), dim3(256), 0, st, N, (double)sigma, p->Wg);
  float *absr = reinterpret_cast<float *>(p->F);   // N^3 floats fit in F
  hipLaunchKernelGGL(abs_kernel, pgrid(n3), dim3(256), 0, st, rho, n3, absr);
  hipError_t e = launch_contract_rows(absr, false, p->Wg, p->T1, N * N, N, N, st);
  if (e == hipSuccess) e = launch_contract(p->T1, p->Wg, p->T2, false, N, N, N, N, st);
  if (e == hipSuccess) e = launch_contract(p->T2, p->Wg, b, true, 1, N, N, N * N, st);
  if (e != hipSuccess) return hip_fail(e, "phase_shrinkwrap: launch");
  hipLaunchKernelGGL(max_partial_kernel, dim3(kPhBlocks), dim3(256), 0, st, b, n3, p->part);
  hipLaunchKernelGGL(threshold_kernel, pgrid(n3), dim3(256), 0, st, b, n3, p->part, tau, support);
  e = hipGetLastError();
  return e == hipSuccess ? SPFEL_OK : hip_fail(e, "phase_shrinkwrap: launch");
}

}  // extern "C"
