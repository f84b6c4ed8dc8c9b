// Regularised merging (section II-C, Eq. (2)):
//   (A* D A + lambda I) x = A* D b + lambda x0,
// with A* D A applied as a convolution on the Cartesian grid (the Toeplitz
// method): (A* D A)_{k k'} = T[k - k'], T the type-1 transform of the
// weights D on (2N - 1)^3 modes (REAL domain: A^T D A x = C * even(x), C the
// cosine transform of D).  On a grid of L = 2N cells per axis the circular
// convolution equals the linear one for |k - k'| <= N - 1 < L / 2, so one
// application is three separable line transforms N -> L, a pointwise
// product with the transformed kernel, and three line transforms L -> N.
// REAL domain: the first line transform reads the even part of the vector (a
// line and the line of the opposite modes); its transform is real and
// Hermitian, so axis 2 keeps its nonnegative half, and what rounding leaves in
// the imaginary parts is dropped before the product.
// Conjugate gradients solve up to kMaxSystems systems (one per lambda) at
// once, sharing every transform launch; the step sizes stay on the device.
#include <cmath>
#include <mutex>
#include <new>
#include <set>
#include <string>
#include <vector>

#include "dft.h"
#include "internal.h"

namespace spfel {

constexpr int kMaxSystems = 16;
constexpr int kDotBlocks = 256;
constexpr int64_t kGroupBytes = (int64_t)208 << 20;

struct Lambdas {
  float v[kMaxSystems];
};

struct Normal {
  int device = 0, N = 0, L = 0, domain = SPFEL_REAL, max_sys = 0;
  int group = 1;           // systems per transform launch
  int Lh = 0;              // cells kept along axis 2: N + 1 (REAL) or L
  DftTable F;              // modes -> grid, exp(-2 pi i k l / L)
  DftTable G;              // grid -> modes, exp(+2 pi i k l / L) / L
  DftTable Hm;             // the 2N - 1 modes of the kernel -> grid, as F
  float2 *That = nullptr;  // [L][L][Lh]: transform of the Toeplitz kernel
  // transform intermediates of a group, [group][N][N][Lh] and
  // [group][N][L][Lh] (X3, [group][L][L][Lh],
  // only where the fused axis-0 pass does not fit the LDS)
  float2 *X1 = nullptr, *X2 = nullptr, *X3 = nullptr;
  void *x = nullptr, *r = nullptr, *p = nullptr, *Ap = nullptr;
  float *scal = nullptr;   // per system: r.r of even and of odd steps, alpha, spare (or lcurve's dots)
  float *part = nullptr;   // two sets of dot partial sums
  bool psf_set = false;
  size_t bytes = 0;
};

static std::mutex g_nmu;
static std::set<Normal *> g_nlive;

static bool nlive(Normal *p) {
  std::lock_guard<std::mutex> lk(g_nmu);
  return p && g_nlive.count(p) > 0;
}

static void free_normal(Normal *p) {
  void *bufs[] = {p->F.t, p->G.t, p->Hm.t, p->That, p->X1, p->X2, p->X3,
                  p->x, p->r, p->p, p->Ap, p->scal, p->part};
  for (void *b : bufs)
    if (b) (void)hipFree(b);
}

// ---------------------------------------------------------------- kernels --

// X[s][j] *= That[j] (complex), j < L3; drop_im: the imaginary part of X is
// dropped first.
__global__ __launch_bounds__(256) void kernel_product(float2 *__restrict__ X,
                                                      const float2 *__restrict__ T, int64_t L3,
                                                      int n, int drop_im) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * L3) return;
  float2 a = X[t];
  const float2 b = T[t % L3];
  if (drop_im)
    X[t] = make_float2(a.x * b.x, a.x * b.y);
  else
    X[t] = make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// Partial sums of sum_k u[s][k] v[k'] (real parts of conj(u) v for complex
// vectors stored as float pairs: the float-pair dot is exactly that), fixed
// order: block b of system s takes a contiguous range, 256 strided partials,
// a pairwise tree.  v_stride 0 broadcasts one vector to every system.
__global__ __launch_bounds__(256) void dot_partial_kernel(const float *__restrict__ u,
                                                          const float *__restrict__ v,
                                                          int64_t len, int64_t v_stride,
                                                          float *__restrict__ part) {
  __shared__ float sh[256];
  const int s = blockIdx.y;
  const int64_t per = (len + kDotBlocks - 1) / kDotBlocks;
  const int64_t lo = (int64_t)blockIdx.x * per, hi = min(len, lo + per);
  const float *us = u + s * len, *vs = v + s * v_stride;
  float acc = 0.f;
#pragma unroll 4
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256) acc = fmaf(us[i], vs[i], acc);
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[s * kDotBlocks + blockIdx.x] = sh[0];
}

// out[s * stride] = sum of the system's partials in block order.
__global__ void dot_final_kernel(const float *__restrict__ part, int n, float *__restrict__ out,
                                 int stride) {
  const int s = threadIdx.x;
  if (s >= n) return;
  float t = 0.f;
  for (int b = 0; b < kDotBlocks; ++b) t += part[s * kDotBlocks + b];
  out[s * stride] = t;
}

// Vector passes of CG: block (b, s) takes the b-th contiguous range of system
// s and leaves its part of a dot product (256 strided sums, a pairwise tree)
// in part[s][b]; every block of the next pass adds the system's parts itself,
// in one fixed order, so no pass of its own forms a step size.
__device__ inline float block_sum(float v, float *sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
    __syncthreads();
  }
  const float t = sh[0];
  __syncthreads();
  return t;
}
static_assert(kDotBlocks == 256, "one part per thread");

// r = p = rhs - A* D A x0 (the lambda terms cancel, so every system starts
// from the same residual), x = x0; part: r.r.
__global__ __launch_bounds__(256) void cg_init_kernel(const float *__restrict__ rhs,
                                                      const float *__restrict__ x0,
                                                      const float *__restrict__ Ax0, int64_t len,
                                                      float *__restrict__ x, float *__restrict__ r,
                                                      float *__restrict__ p,
                                                      float *__restrict__ part) {
  __shared__ float sh[256];
  const int s = blockIdx.y;
  const int64_t per = (len + kDotBlocks - 1) / kDotBlocks;
  const int64_t lo = (int64_t)blockIdx.x * per, hi = min(len, lo + per);
  x += s * len;
  r += s * len;
  p += s * len;
  float acc = 0.f;
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
    const float v = rhs[i] - Ax0[i];
    x[i] = x0[i];
    r[i] = v;
    p[i] = v;
    acc = fmaf(v, v, acc);
  }
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) part[s * kDotBlocks + blockIdx.x] = acc;
}

// scal[s][0] = r.r of the start; hist[s][0] = |r|.
__global__ __launch_bounds__(256) void cg_start_kernel(const float *__restrict__ part,
                                                       float *__restrict__ scal,
                                                       float *__restrict__ hist, int stride) {
  __shared__ float sh[256];
  const int s = blockIdx.x;
  const float rr = block_sum(part[s * kDotBlocks + threadIdx.x], sh);
  if (threadIdx.x == 0) {
    scal[4 * s] = rr;
    if (hist) hist[s * stride] = sqrtf(fmaxf(rr, 0.f));
  }
}

// alpha = rr / p.Ap (0 once converged), r -= alpha Ap; part_rr: r.r.  scal[s]:
// rr of the even and of the odd steps, alpha.
__global__ __launch_bounds__(256) void cg_residual_kernel(const float *__restrict__ part_pAp,
                                                          float *__restrict__ scal, int it,
                                                          const float *__restrict__ Ap, int64_t len,
                                                          float *__restrict__ r,
                                                          float *__restrict__ part_rr) {
  __shared__ float sh[256];
  const int s = blockIdx.y;
  const float pAp = block_sum(part_pAp[s * kDotBlocks + threadIdx.x], sh);
  const float rr = scal[4 * s + ((it - 1) & 1)];
  const float alpha = pAp > 0.f && rr > 0.f ? rr / pAp : 0.f;
  if (blockIdx.x == 0 && threadIdx.x == 0) scal[4 * s + 2] = alpha;
  const int64_t per = (len + kDotBlocks - 1) / kDotBlocks;
  const int64_t lo = (int64_t)blockIdx.x * per, hi = min(len, lo + per);
  r += s * len;
  Ap += s * len;
  float acc = 0.f;
#pragma unroll 4
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
    const float v = fmaf(-alpha, Ap[i], r[i]);
    r[i] = v;
    acc = fmaf(v, v, acc);
  }
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) part_rr[s * kDotBlocks + blockIdx.x] = acc;
}

// beta = rr_new / rr; x += alpha p, p = r + beta p; hist[s][it] = |r|.
__global__ __launch_bounds__(256) void cg_direction_kernel(const float *__restrict__ part_rr,
                                                           float *__restrict__ scal, int it,
                                                           const float *__restrict__ r, int64_t len,
                                                           float *__restrict__ x,
                                                           float *__restrict__ p,
                                                           float *__restrict__ hist, int stride) {
  __shared__ float sh[256];
  const int s = blockIdx.y;
  const float rr_new = block_sum(part_rr[s * kDotBlocks + threadIdx.x], sh);
  const float rr = scal[4 * s + ((it - 1) & 1)], alpha = scal[4 * s + 2];
  const float beta = rr > 0.f ? rr_new / rr : 0.f;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    scal[4 * s + (it & 1)] = rr_new;
    if (hist) hist[s * stride + it] = sqrtf(fmaxf(rr_new, 0.f));
  }
  const int64_t per = (len + kDotBlocks - 1) / kDotBlocks;
  const int64_t lo = (int64_t)blockIdx.x * per, hi = min(len, lo + per);
  r += s * len;
  x += s * len;
  p += s * len;
#pragma unroll 4
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
    const float v = p[i];
    x[i] = fmaf(alpha, v, x[i]);
    p[i] = fmaf(beta, v, r[i]);
  }
}

// d = x - x0 (x0 shared).
__global__ __launch_bounds__(256) void diff_kernel(const float *__restrict__ x,
                                                   const float *__restrict__ x0, int64_t len,
                                                   int n, float *__restrict__ d) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * len) return;
  d[t] = x[t] - x0[t % len];
}

// rho = x.Hx - 2 x.rhs + bdb, eta = |x - x0|^2 from the dots (scal[s][0..2]
// = x.Hx, x.rhs, eta); corner of the L-curve by the largest curvature of
// (log rho, log eta) over log lambda (central differences, end points
// excluded; uniform spacing in log lambda assumed).
__global__ void lcurve_kernel(const float *__restrict__ scal, int n, double bdb, Lambdas lam,
                              float *__restrict__ rho_eta, int32_t *__restrict__ corner) {
  if (threadIdx.x != 0) return;
  double u[kMaxSystems], v[kMaxSystems];
  for (int s = 0; s < n; ++s) {
    const double rho = (double)scal[4 * s] - 2.0 * (double)scal[4 * s + 1] + bdb;
    const double eta = (double)scal[4 * s + 2];
    rho_eta[2 * s] = (float)rho;
    rho_eta[2 * s + 1] = (float)eta;
    u[s] = log(fmax(rho, 1e-300));
    v[s] = log(fmax(eta, 1e-300));
  }
  if (!corner) return;
  int arg = n > 2 ? 1 : 0;
  if (n > 2) {
    const double dt = log((double)lam.v[1]) - log((double)lam.v[0]);
    double best = -1e300;
    for (int i = 1; i < n - 1; ++i) {
      const double du = (u[i + 1] - u[i - 1]) / (2 * dt), dv = (v[i + 1] - v[i - 1]) / (2 * dt);
      const double ddu = (u[i + 1] - 2 * u[i] + u[i - 1]) / (dt * dt);
      const double ddv = (v[i + 1] - 2 * v[i] + v[i - 1]) / (dt * dt);
      const double kappa = (du * ddv - ddu * dv) / pow(du * du + dv * dv, 1.5);
      if (kappa > best) {
        best = kappa;
        arg = i;
      }
    }
  }
  *corner = arg;
}

static dim3 grid_of(int64_t n) { return dim3((unsigned)((n + 255) / 256)); }

// y[s] = A* D A v[s] (+ lambda_s v[s]) for s < n.
static hipError_t normal_apply(const Normal &nm, const void *v, int n, const Lambdas *lam,
                               void *y, hipStream_t st) {
  if (n > nm.group) {   // in groups whose intermediates stay in the memory-side cache
    const size_t vec = (size_t)nm.N * nm.N * nm.N * (nm.domain == SPFEL_COMPLEX ? 8 : 4);
    for (int s0 = 0; s0 < n; s0 += nm.group) {
      const int m = n - s0 < nm.group ? n - s0 : nm.group;
      Lambdas part{};
      for (int s = 0; lam && s < m; ++s) part.v[s] = lam->v[s0 + s];
      hipError_t e = normal_apply(nm, static_cast<const char *>(v) + s0 * vec, m, lam ? &part : nullptr,
                                  static_cast<char *>(y) + s0 * vec, st);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  const int64_t N = nm.N, L = nm.L, Lh = nm.Lh;
  const bool cplx = nm.domain == SPFEL_COMPLEX;
  const int64_t cols = L * Lh;
  DftEpilogue first, none, last;
  first.even_lines = cplx ? 0 : N * N;
  hipError_t e = launch_dft(nm.F, cplx ? kCC : kRH, {n * N * N, 1, (int)N, (int)Lh}, v, nm.X1, first, st);
  if (e == hipSuccess)
    e = launch_dft(nm.F, kCC, {n * N * Lh, (int)Lh, (int)N, (int)L}, nm.X1, nm.X2, none, st);
  if (e != hipSuccess) return e;
  if (!nm.X3) {
    e = launch_dft_normal(nm.F, nm.G, cplx, nm.X2, nm.That, n, cols, st);
  } else {
    e = launch_dft(nm.F, kCC, {n * cols, (int)cols, (int)N, (int)L}, nm.X2, nm.X3, none, st);
    hipLaunchKernelGGL(kernel_product, grid_of(n * L * cols), dim3(256), 0, st, nm.X3, nm.That,
                       L * cols, n, cplx ? 0 : 1);
    if (e == hipSuccess)
      e = launch_dft(nm.G, kCC, {n * cols, (int)cols, (int)L, (int)N}, nm.X3, nm.X2, none, st);
  }
  if (e == hipSuccess)
    e = launch_dft(nm.G, kCC, {n * N * Lh, (int)Lh, (int)L, (int)N}, nm.X2, nm.X1, none, st);
  if (e != hipSuccess) return e;
  if (lam) {
    last.lam_v = v;
    last.lambda = lam->v;
    last.systems = n;
    last.cols_per_system = N * N;
  }
  return launch_dft(nm.G, cplx ? kCC : kHR, {n * N * N, 1, (int)Lh, (int)N}, nm.X1, y, last, st);
}

// out[s * stride] = u[s] . v[s or shared], over len floats.
static hipError_t dots(const Normal &nm, const void *u, const void *v, int64_t len,
                       int64_t v_stride, int n, float *out, int stride, hipStream_t st) {
  hipLaunchKernelGGL(dot_partial_kernel, dim3(kDotBlocks, n), dim3(256), 0, st,
                     static_cast<const float *>(u), static_cast<const float *>(v), len, v_stride,
                     nm.part);
  hipLaunchKernelGGL(dot_final_kernel, dim3(1), dim3(64), 0, st, nm.part, n, out, stride);
  return hipGetLastError();
}

}  // namespace spfel

using namespace spfel;

extern "C" {

int spfel_normal_create(spfel_normal *out, int n_model, int domain, int max_systems,
                        int device) {
  clear_error();
  if (!out) return fail(SPFEL_EINVAL, "normal_create: out is NULL");
  *out = nullptr;
  if (n_model < 3 || n_model % 2 == 0) return fail(SPFEL_EINVAL, "normal_create: n_model must be odd and >= 3");
  if (n_model > 511) return fail(SPFEL_ERANGE, "normal_create: n_model > 511");
  if (domain != SPFEL_REAL && domain != SPFEL_COMPLEX)
    return fail(SPFEL_EINVAL, "normal_create: domain must be REAL or COMPLEX");
  if (max_systems < 1 || max_systems > kMaxSystems)
    return fail(SPFEL_EINVAL, "normal_create: max_systems must be 1..16");
  int ndev = 0;
  hipError_t e = hipGetDeviceCount(&ndev);
  if (e != hipSuccess) return hip_fail(e, "normal_create: hipGetDeviceCount");
  if (device < 0 || device >= ndev) return fail(SPFEL_EINVAL, "normal_create: no such device");
  int prev = 0;
  (void)hipGetDevice(&prev);
  if (prev != device) (void)hipSetDevice(device);
  Normal *p = new (std::nothrow) Normal();
  if (!p) return fail(SPFEL_ENOMEM, "normal_create: host allocation");
  p->device = device;
  p->N = n_model;
  p->L = 2 * n_model;
  p->domain = domain;
  p->max_sys = max_systems;
  const int64_t N = n_model, L = p->L, M = 2 * N - 1, n = max_systems;
  const int64_t N3 = N * N * N, L3 = L * L * L;
  const size_t vec = (size_t)N3 * (domain == SPFEL_COMPLEX ? 8 : 4);
  const int64_t Lh = domain == SPFEL_COMPLEX ? L : N + 1, cols = L * Lh;
  p->Lh = (int)Lh;
  // systems per launch: their intermediates together about the memory-side
  // cache (256 MB; 8 systems at N = 129 in groups of 2 / 4 / 8: 3.78 / 3.54 /
  // 3.64 ms for three CG steps)
  const int64_t per_system = (N * N * Lh + N * L * Lh) * 8;
  p->group = (int)std::max<int64_t>(1, std::min<int64_t>(n, kGroupBytes / per_system));
  const int64_t gr = p->group;
  const size_t tab_f = dft_table_sizes(p->F, kToGrid, (n_model - 1) / 2, n_model);
  const size_t tab_g = dft_table_sizes(p->G, kToModes, (n_model - 1) / 2, n_model);
  const size_t tab_h = dft_table_sizes(p->Hm, kToGrid, n_model - 1, n_model);
  const bool fused = dft_normal_fits(p->F, p->G, domain == SPFEL_COMPLEX);
  struct Req {
    void **ptr;
    size_t bytes;
  } reqs[] = {{reinterpret_cast<void **>(&p->F.t), tab_f},
              {reinterpret_cast<void **>(&p->G.t), tab_g},
              {reinterpret_cast<void **>(&p->Hm.t), tab_h},
              {reinterpret_cast<void **>(&p->That), (size_t)(L * cols) * 8},
              {reinterpret_cast<void **>(&p->X1), (size_t)std::max(gr * N * N * Lh, M * M * Lh) * 8},
              {reinterpret_cast<void **>(&p->X2), (size_t)std::max(gr * N * cols, M * cols) * 8},
              {reinterpret_cast<void **>(&p->X3), fused ? 0 : (size_t)(gr * L * cols) * 8},
              {&p->x, n * vec},
              {&p->r, n * vec},
              {&p->p, n * vec},
              {&p->Ap, n * vec},
              {reinterpret_cast<void **>(&p->scal), (size_t)kMaxSystems * 4 * 4},
              {reinterpret_cast<void **>(&p->part), 2 * (size_t)kMaxSystems * kDotBlocks * 4}};
  for (auto &r : reqs) {
    if (r.bytes == 0) continue;
    e = hipMalloc(r.ptr, r.bytes);
    if (e != hipSuccess) {
      *r.ptr = nullptr;
      (void)hipGetLastError();
      free_normal(p);
      delete p;
      if (prev != device) (void)hipSetDevice(prev);
      return fail(SPFEL_ENOMEM, std::string("normal_create: hipMalloc: ") + hipGetErrorString(e));
    }
    p->bytes += r.bytes;
  }
  const double scale = 1.0 / (double)L;
  e = dft_table_fill(p->F, -1, [](int) { return 1.0; });
  if (e == hipSuccess) e = dft_table_fill(p->G, +1, [&](int) { return scale; });
  if (e == hipSuccess) e = dft_table_fill(p->Hm, -1, [](int) { return 1.0; });
  if (prev != device) (void)hipSetDevice(prev);
  if (e != hipSuccess) {
    free_normal(p);
    delete p;
    return hip_fail(e, "normal_create: table upload");
  }
  {
    std::lock_guard<std::mutex> lk(g_nmu);
    g_nlive.insert(p);
  }
  *out = reinterpret_cast<spfel_normal>(p);
  return SPFEL_OK;
}

int spfel_normal_destroy(spfel_normal h) {
  clear_error();
  Normal *p = reinterpret_cast<Normal *>(h);
  {
    std::lock_guard<std::mutex> lk(g_nmu);
    if (!p || g_nlive.erase(p) == 0) return fail(SPFEL_ESTATE, "normal_destroy: not a live object");
  }
  free_normal(p);
  delete p;
  return SPFEL_OK;
}

int spfel_normal_set_psf(spfel_normal h, const void *psf, void *stream) {
  clear_error();
  Normal *p = reinterpret_cast<Normal *>(h);
  if (!nlive(p)) return fail(SPFEL_ESTATE, "normal_set_psf: not a live object");
  if (!psf) return fail(SPFEL_EINVAL, "normal_set_psf: psf is NULL");
  const bool cplx = p->domain == SPFEL_COMPLEX;
  if ((reinterpret_cast<uintptr_t>(psf) & (cplx ? 7 : 3)) != 0)
    return fail(SPFEL_EINVAL, "normal_set_psf: psf misaligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int64_t M = 2 * p->N - 1, L = p->L, Lh = p->Lh;
  // That = DFT_L of the kernel placed at m mod L: three line transforms M -> L
  const DftEpilogue none;
  hipError_t e = launch_dft(p->Hm, cplx ? kCC : kRH, {M * M, 1, (int)M, (int)Lh}, psf, p->X1, none, st);
  if (e == hipSuccess)
    e = launch_dft(p->Hm, kCC, {M * Lh, (int)Lh, (int)M, (int)L}, p->X1, p->X2, none, st);
  if (e == hipSuccess)
    e = launch_dft(p->Hm, kCC, {L * Lh, (int)(L * Lh), (int)M, (int)L}, p->X2, p->That, none, st);
  if (e != hipSuccess) return hip_fail(e, "normal_set_psf: launch");
  p->psf_set = true;
  return SPFEL_OK;
}

// Vectors are float32 (REAL) or complex64 (COMPLEX) arrays.
static bool vec_aligned(const Normal *p, const void *v) {
  return (reinterpret_cast<uintptr_t>(v) & (p->domain == SPFEL_COMPLEX ? 7 : 3)) == 0;
}

static int check_lambdas(const Normal *p, int n, const float *lambdas, Lambdas &lam,
                         const char *who) {
  if (n < 1 || n > p->max_sys) return fail(SPFEL_EINVAL, std::string(who) + ": n out of 1..max_systems");
  if (!lambdas) return fail(SPFEL_EINVAL, std::string(who) + ": lambdas is NULL");
  for (int s = 0; s < kMaxSystems; ++s) lam.v[s] = 0.f;
  for (int s = 0; s < n; ++s) {
    if (!(lambdas[s] >= 0.f) || !std::isfinite(lambdas[s]))
      return fail(SPFEL_EINVAL, std::string(who) + ": lambdas must be finite and >= 0");
    lam.v[s] = lambdas[s];
  }
  return SPFEL_OK;
}

int spfel_normal_apply(spfel_normal h, const void *x, int n, const float *lambdas, void *y,
                       void *stream) {
  clear_error();
  Normal *p = reinterpret_cast<Normal *>(h);
  if (!nlive(p)) return fail(SPFEL_ESTATE, "normal_apply: not a live object");
  if (!p->psf_set) return fail(SPFEL_ESTATE, "normal_apply: set_psf has not been called");
  Lambdas lam;
  int rc = check_lambdas(p, n, lambdas, lam, "normal_apply");
  if (rc != SPFEL_OK) return rc;
  if (!x || !y) return fail(SPFEL_EINVAL, "normal_apply: NULL pointer");
  if (!vec_aligned(p, x) || !vec_aligned(p, y)) return fail(SPFEL_EINVAL, "normal_apply: misaligned vector");
  hipError_t e = normal_apply(*p, x, n, &lam, y, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? SPFEL_OK : hip_fail(e, "normal_apply: launch");
}

int spfel_normal_solve(spfel_normal h, const void *rhs, const void *x0, int n,
                       const float *lambdas, int iters, void *x_out, float *residuals,
                       void *stream) {
  clear_error();
  Normal *p = reinterpret_cast<Normal *>(h);
  if (!nlive(p)) return fail(SPFEL_ESTATE, "normal_solve: not a live object");
  if (!p->psf_set) return fail(SPFEL_ESTATE, "normal_solve: set_psf has not been called");
  Lambdas lam;
  int rc = check_lambdas(p, n, lambdas, lam, "normal_solve");
  if (rc != SPFEL_OK) return rc;
  if (!rhs || !x0 || !x_out) return fail(SPFEL_EINVAL, "normal_solve: NULL pointer");
  if (!vec_aligned(p, rhs) || !vec_aligned(p, x0) || !vec_aligned(p, x_out) ||
      (reinterpret_cast<uintptr_t>(residuals) & 3))
    return fail(SPFEL_EINVAL, "normal_solve: misaligned vector");
  if (iters < 0 || iters > 100000) return fail(SPFEL_EINVAL, "normal_solve: iters out of 0..100000");
  hipStream_t st = static_cast<hipStream_t>(stream);
  const bool cplx = p->domain == SPFEL_COMPLEX;
  const int64_t N3 = (int64_t)p->N * p->N * p->N, len = N3 * (cplx ? 2 : 1);
  const float *rf = static_cast<const float *>(rhs), *x0f = static_cast<const float *>(x0);
  float *xf = static_cast<float *>(x_out), *r = static_cast<float *>(p->r);
  float *pp = static_cast<float *>(p->p), *Ap = static_cast<float *>(p->Ap);
  const int stride = iters + 1;
  const dim3 vec(kDotBlocks, (unsigned)n);
  float *part_rr = p->part + kMaxSystems * kDotBlocks;
  // A* D A x0 once: r = rhs + lambda x0 - (A* D A + lambda) x0 for every lambda
  hipError_t e = normal_apply(*p, x0f, 1, nullptr, Ap, st);
  if (e != hipSuccess) return hip_fail(e, "normal_solve: launch");
  hipLaunchKernelGGL(cg_init_kernel, vec, dim3(256), 0, st, rf, x0f, Ap, len, xf, r, pp, part_rr);
  hipLaunchKernelGGL(cg_start_kernel, dim3((unsigned)n), dim3(256), 0, st, part_rr, p->scal, residuals,
                     stride);
  for (int it = 1; it <= iters; ++it) {
    e = normal_apply(*p, pp, n, &lam, Ap, st);
    if (e != hipSuccess) return hip_fail(e, "normal_solve: launch");
    hipLaunchKernelGGL(dot_partial_kernel, vec, dim3(256), 0, st, pp, Ap, len, len, p->part);
    hipLaunchKernelGGL(cg_residual_kernel, vec, dim3(256), 0, st, p->part, p->scal, it, Ap, len, r,
                       part_rr);
    hipLaunchKernelGGL(cg_direction_kernel, vec, dim3(256), 0, st, part_rr, p->scal, it, r, len, xf,
                       pp, residuals, stride);
  }
  e = hipGetLastError();
  return e == hipSuccess ? SPFEL_OK : hip_fail(e, "normal_solve: launch");
}

int spfel_normal_lcurve(spfel_normal h, const void *x, const void *rhs, const void *x0, int n,
                        const float *lambdas, double bdb, float *rho_eta, int32_t *corner,
                        void *stream) {
  clear_error();
  Normal *p = reinterpret_cast<Normal *>(h);
  if (!nlive(p)) return fail(SPFEL_ESTATE, "normal_lcurve: not a live object");
  if (!p->psf_set) return fail(SPFEL_ESTATE, "normal_lcurve: set_psf has not been called");
  Lambdas lam;
  int rc = check_lambdas(p, n, lambdas, lam, "normal_lcurve");
  if (rc != SPFEL_OK) return rc;
  if (!x || !rhs || !x0 || !rho_eta) return fail(SPFEL_EINVAL, "normal_lcurve: NULL pointer");
  if (!vec_aligned(p, x) || !vec_aligned(p, rhs) || !vec_aligned(p, x0) ||
      (reinterpret_cast<uintptr_t>(rho_eta) & 3) || (reinterpret_cast<uintptr_t>(corner) & 3))
    return fail(SPFEL_EINVAL, "normal_lcurve: misaligned array");
  if (n >= 3)
    for (int s = 0; s < n; ++s)
      if (!(lambdas[s] > 0.f))
        return fail(SPFEL_EINVAL, "normal_lcurve: the corner needs lambdas > 0 (log spacing)");
  hipStream_t st = static_cast<hipStream_t>(stream);
  const bool cplx = p->domain == SPFEL_COMPLEX;
  const int64_t N3 = (int64_t)p->N * p->N * p->N, len = N3 * (cplx ? 2 : 1);
  // Ap = A* D A x (no lambda); scal[s] = (x.Ap, x.rhs, |x - x0|^2)
  hipError_t e = normal_apply(*p, x, n, nullptr, p->Ap, st);
  if (e == hipSuccess) e = dots(*p, x, p->Ap, len, len, n, p->scal, 4, st);
  if (e == hipSuccess) e = dots(*p, x, rhs, len, 0, n, p->scal + 1, 4, st);
  if (e != hipSuccess) return hip_fail(e, "normal_lcurve: launch");
  hipLaunchKernelGGL(diff_kernel, grid_of(n * len), dim3(256), 0, st,
                     static_cast<const float *>(x), static_cast<const float *>(x0), len, n,
                     static_cast<float *>(p->r));
  e = dots(*p, p->r, p->r, len, len, n, p->scal + 2, 4, st);
  if (e != hipSuccess) return hip_fail(e, "normal_lcurve: launch");
  hipLaunchKernelGGL(lcurve_kernel, dim3(1), dim3(64), 0, st, p->scal, n, bdb, lam, rho_eta,
                     corner);
  e = hipGetLastError();
  return e == hipSuccess ? SPFEL_OK : hip_fail(e, "normal_lcurve: launch");
}

}  // extern "C"
