// DOS reconstructions from Chebyshev moments, FP64 throughout.
//
// KPM (paper eqs. e7 and delta_function_cheb_expansion) with a damping kernel:
//   rho(E) = [g_0 mu_0 + 2 sum_{n>=1} g_n mu_n T_n(eps)] / (pi sqrt(1 - eps^2) de-),
// g_n the Jackson kernel (Weisse et al. 2006, which the paper cites) or the
// Lorentz kernel the paper prints (Sec. 2(a)).  One workgroup stages
// c_n = g_n mu_n (x2 for n >= 1) in LDS in chunks; each thread owns one energy
// and runs the scalar Chebyshev recursion in eps.
//
// CPGF (eqs. green_function_cheb_expansion(b)): the retarded resolvent
//   (1/N) Tr 1/(E - H + i eta) = (1/de-) sum_n g_n(z) mu_n / (1 + delta_n0),
//   g_n(z) = -2 i w^n / sqrt(1 - z^2),  z = eps + i eta/de-,  w = exp(-i arccos z).
// w is the root of w^2 - 2 z w + 1 = 0 inside the unit circle (taken as the
// reciprocal of the outer root, which has no cancellation), and with that
// branch sqrt(1 - z^2) = i (w - z), so g_n = -2 w^n / (w - z).

#include "kpm_internal.h"
#include "kpm_stencil.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

namespace kpm {

enum { kKernelJackson = 0, kKernelLorentz = 1 };

__device__ inline double damping(int kernel, int n, int M, double lam) {
  if (kernel == kKernelLorentz) return sinh(lam * (1.0 - (double)n / M)) / sinh(lam);
  const double q = M_PI / (M + 1);
  return ((M - n + 1) * cos(q * n) + sin(q * n) / tan(q)) / (M + 1);
}

__global__ void kernel_dos_kernel(const double* mu, int M, const double* energies, int K, double e_min,
                                  double e_max, int kernel, double lam, double* rho) {
  __shared__ double coef[1024];
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const double de_p = 0.5 * (e_max + e_min), de_m = 0.5 * (e_max - e_min);
  const double eps = (k < K) ? (energies[k] - de_p) / de_m : 0.0;
  const bool inside = (k < K) && fabs(eps) < 1.0;
  double tm1 = 1.0, t0 = eps, acc = 0.0;   // T_{n-1}, T_n as the recursion advances
  for (int base = 0; base < M; base += 1024) {
    __syncthreads();
    for (int i = threadIdx.x; i < 1024 && base + i < M; i += blockDim.x) {
      const int n = base + i;
      coef[i] = (n == 0 ? 1.0 : 2.0) * damping(kernel, n, M, lam) * mu[n];
    }
    __syncthreads();
    const int cnt = min(1024, M - base);
    for (int i = 0; i < cnt; ++i) {
      const int n = base + i;
      double tn;
      if (n == 0) tn = 1.0;
      else if (n == 1) tn = eps;
      else {
        tn = 2.0 * eps * t0 - tm1;
        tm1 = t0;
        t0 = tn;
      }
      acc += coef[i] * tn;
    }
  }
  if (k < K) rho[k] = inside ? acc / (M_PI * sqrt(1.0 - eps * eps) * de_m) : 0.0;
}

struct cplx {
  double re, im;
};
__device__ inline cplx cmul(cplx a, cplx b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ inline cplx cdiv(cplx a, cplx b) {
  // Smith's algorithm (scaled by the larger component of b).
  if (fabs(b.re) >= fabs(b.im)) {
    const double r = b.im / b.re, d = b.re + b.im * r;
    return {(a.re + a.im * r) / d, (a.im - a.re * r) / d};
  }
  const double r = b.re / b.im, d = b.re * r + b.im;
  return {(a.re * r + a.im) / d, (a.im * r - a.re) / d};
}
// Principal square root.
__device__ inline cplx csqrt_p(cplx z) {
  const double m = hypot(z.re, z.im);
  if (m == 0.0) return {0.0, 0.0};
  if (z.re >= 0.0) {
    const double p = sqrt(0.5 * (m + z.re));
    return {p, z.im / (2.0 * p)};
  }
  const double q = copysign(sqrt(0.5 * (m - z.re)), z.im);
  return {z.im / (2.0 * q), q};
}

__global__ void cpgf_kernel(const double* mu, int M, const double* energies, int K, double e_min, double e_max,
                            double eta_ev, double* rho, double* green) {
  __shared__ double cm[1024];
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const double de_p = 0.5 * (e_max + e_min), de_m = 0.5 * (e_max - e_min);
  const cplx z = {(k < K) ? (energies[k] - de_p) / de_m : 0.0, eta_ev / de_m};
  // Roots of w^2 - 2 z w + 1: z +- sqrt(z^2 - 1); the outer one has |.| > 1.
  const cplx s = csqrt_p({z.re * z.re - z.im * z.im - 1.0, 2.0 * z.re * z.im});
  const cplx wp = {z.re + s.re, z.im + s.im}, wm = {z.re - s.re, z.im - s.im};
  const cplx outer = (hypot(wp.re, wp.im) >= hypot(wm.re, wm.im)) ? wp : wm;
  const cplx w = cdiv({1.0, 0.0}, outer);
  cplx pw = {1.0, 0.0};   // w^n
  cplx acc = {0.0, 0.0};  // sum_n mu_n w^n / (1 + delta_n0)
  for (int base = 0; base < M; base += 1024) {
    __syncthreads();
    for (int i = threadIdx.x; i < 1024 && base + i < M; i += blockDim.x) {
      const int n = base + i;
      cm[i] = (n == 0 ? 0.5 : 1.0) * mu[n];
    }
    __syncthreads();
    const int cnt = min(1024, M - base);
    for (int i = 0; i < cnt; ++i) {
      acc.re += cm[i] * pw.re;
      acc.im += cm[i] * pw.im;
      pw = cmul(pw, w);
    }
  }
  // G = -2 acc / ((w - z) de-).
  const cplx g = cdiv({-2.0 * acc.re / de_m, -2.0 * acc.im / de_m}, {w.re - z.re, w.im - z.im});
  if (k < K) {
    rho[k] = -g.im / M_PI;
    if (green) {
      green[2 * k] = g.re;
      green[2 * k + 1] = g.im;
    }
  }
}

// T=0 longitudinal conductivity from Gamma (Kubo-Greenwood limit of the
// first-order formula, with eq. delta_function_cheb_expansion for both deltas):
//   sigma(E) = -2 pi^2 (N/Omega) / de-^2  sum_nm g_n g_m D_n(eps) D_m(eps) Re Gamma_nm   [e^2/h],
//   D_n(eps) = 2 T_n(eps) / (pi sqrt(1 - eps^2)).
// One workgroup per energy; w_n = g_n D_n(eps) staged in LDS.
__global__ void sigma_kernel(const double* gamma, int M, const double* energies, int K, double e_min, double e_max,
                             double density, double* sigma) {
  extern __shared__ double w[];
  __shared__ double red[256];
  const int k = blockIdx.x;
  const double de_p = 0.5 * (e_max + e_min), de_m = 0.5 * (e_max - e_min);
  const double eps = (energies[k] - de_p) / de_m;
  if (!(fabs(eps) < 1.0)) {
    if (threadIdx.x == 0) sigma[k] = 0.0;
    return;
  }
  const double th = acos(eps);
  const double pref = 2.0 / (M_PI * sqrt(1.0 - eps * eps));
  for (int n = threadIdx.x; n < M; n += blockDim.x) w[n] = damping(kKernelJackson, n, M, 0.0) * pref * cos(n * th);
  __syncthreads();
  double acc = 0.0;
  for (int n = threadIdx.x; n < M; n += blockDim.x) {
    const double* row = gamma + (int64_t)n * M * 2;
    double rs = 0.0;
    for (int m = 0; m < M; ++m) rs += row[2 * m] * w[m];
    acc += w[n] * rs;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int st = blockDim.x / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) sigma[k] = -2.0 * M_PI * M_PI * density / (de_m * de_m) * red[0];
}

}  // namespace kpm

extern "C" int kpm_reconstruct_sigma(const double* gamma, int32_t M, const double* energies_ev, int32_t K,
                                     double e_min, double e_max, double orbitals_per_nm2, double* sigma,
                                     int32_t on_device, void* hip_stream) {
  using namespace kpm;
  clear_error();
  KPM_CHECK_ARG(gamma && energies_ev && sigma, "NULL argument");
  KPM_CHECK_ARG(M >= 1 && M <= 8192 && K >= 1, "need 1 <= M <= 8192 and K >= 1");
  KPM_CHECK_ARG(std::isfinite(e_min) && std::isfinite(e_max) && e_min < e_max, "need e_min < e_max");
  KPM_CHECK_ARG(orbitals_per_nm2 > 0.0, "orbitals_per_nm2 must be > 0");
  hipStream_t s = (hipStream_t)hip_stream;
  const double* dg = gamma;
  const double* den = energies_ev;
  double* dsig = sigma;
  double* tmp = nullptr;
  const size_t gn = (size_t)M * M * 2;
  hipError_t e = hipSuccess;
  if (!on_device) {
    e = ::kpm::dev_malloc(&tmp, sizeof(double) * (gn + 2 * (size_t)K));
    if (e == hipSuccess) e = KPM_HIP(hipMemcpyAsync(tmp, gamma, sizeof(double) * gn, hipMemcpyHostToDevice, s));
    if (e == hipSuccess)
      e = KPM_HIP(hipMemcpyAsync(tmp + gn, energies_ev, sizeof(double) * K, hipMemcpyHostToDevice, s));
    dg = tmp;
    den = tmp + gn;
    dsig = tmp + gn + K;
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(sigma_kernel, dim3(K), dim3(256), sizeof(double) * M, s, dg, M, den, K, e_min, e_max,
                       orbitals_per_nm2, dsig);
    e = ::kpm::launch_status();
  }
  if (e == hipSuccess && !on_device) {
    e = hipMemcpyAsync(sigma, dsig, sizeof(double) * K, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
  }
  if (tmp) (void)::kpm::dev_free(tmp, e == hipSuccess);   // (host output: waited for)
  if (e != hipSuccess) {
    set_error("kpm_reconstruct_sigma: %s", hipGetErrorString(e));
    return ::kpm::hip_status(e);
  }
  return KPM_OK;
}

namespace kpm {
// Shared driver: stages host inputs, launches one of the DOS kernels, copies
// the outputs back.  green (CPGF only) may be NULL.
static int reconstruct(const char* name, int which, const double* mu, int32_t M, const double* energies_ev,
                       int32_t K, double e_min, double e_max, double param, double* rho, double* green,
                       int32_t on_device, void* hip_stream) {
  KPM_CHECK_ARG(mu && energies_ev && rho, "NULL argument");
  KPM_CHECK_ARG(M >= 1 && K >= 1, "need M >= 1 and K >= 1");
  KPM_CHECK_ARG(std::isfinite(e_min) && std::isfinite(e_max) && e_min < e_max, "need e_min < e_max");
  hipStream_t s = (hipStream_t)hip_stream;
  const double* dmu = mu;
  const double* den = energies_ev;
  double* drho = rho;
  double* dg = green;
  double* tmp = nullptr;
  hipError_t e = hipSuccess;
  if (!on_device) {
    e = ::kpm::dev_malloc(&tmp, sizeof(double) * ((size_t)M + 4 * (size_t)K));
    if (e == hipSuccess) e = KPM_HIP(hipMemcpyAsync(tmp, mu, sizeof(double) * M, hipMemcpyHostToDevice, s));
    if (e == hipSuccess)
      e = KPM_HIP(hipMemcpyAsync(tmp + M, energies_ev, sizeof(double) * K, hipMemcpyHostToDevice, s));
    dmu = tmp;
    den = tmp + M;
    drho = tmp + M + K;
    dg = green ? tmp + M + 2 * (size_t)K : nullptr;
  }
  if (e == hipSuccess) {
    const dim3 grid((unsigned)ceil_div(K, 256)), block(256);
    if (which == 2)
      hipLaunchKernelGGL(cpgf_kernel, grid, block, 0, s, dmu, M, den, K, e_min, e_max, param, drho, dg);
    else
      hipLaunchKernelGGL(kernel_dos_kernel, grid, block, 0, s, dmu, M, den, K, e_min, e_max, which, param, drho);
    e = ::kpm::launch_status();
  }
  if (e == hipSuccess && !on_device) {
    e = hipMemcpyAsync(rho, drho, sizeof(double) * K, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess && green) e = hipMemcpyAsync(green, dg, sizeof(double) * 2 * K, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
  }
  if (tmp) (void)::kpm::dev_free(tmp, e == hipSuccess);   // (host output: waited for)
  if (e != hipSuccess) {
    set_error("%s: %s", name, hipGetErrorString(e));
    return ::kpm::hip_status(e);
  }
  return KPM_OK;
}
}  // namespace kpm

namespace kpm {
__global__ void kernel_factors_kernel(int kernel, int M, double lam, int n0, int count, double* g) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) g[i] = damping(kernel, n0 + i, M, lam);
}
}  // namespace kpm

extern "C" int kpm_kernel_factors(int32_t kernel, int32_t M, double lambda, int32_t n0, int32_t count, double* g,
                                  int32_t on_device, void* hip_stream) {
  kpm::clear_error();
  KPM_CHECK_ARG(kernel == kpm::kKernelJackson || kernel == kpm::kKernelLorentz, "kernel must be 0 (Jackson) or 1 (Lorentz)");
  KPM_CHECK_ARG(M >= 1 && n0 >= 0 && count >= 1 && (int64_t)n0 + count <= M, "need 0 <= n0 < n0 + count <= M");
  KPM_CHECK_ARG(kernel == kpm::kKernelJackson || (std::isfinite(lambda) && lambda > 0.0), "lambda must be > 0");
  KPM_CHECK_ARG(g != nullptr, "NULL argument");
  hipStream_t s = (hipStream_t)hip_stream;
  double* dg = g;
  if (!on_device) KPM_TRY_HIP(::kpm::dev_malloc(&dg, sizeof(double) * (size_t)count));
  hipLaunchKernelGGL(kpm::kernel_factors_kernel, dim3((unsigned)kpm::ceil_div(count, 256)), dim3(256), 0, s, kernel, M,
                     lambda, n0, count, dg);
  hipError_t e = ::kpm::launch_status();
  if (e == hipSuccess && !on_device) {
    e = hipMemcpyAsync(g, dg, sizeof(double) * (size_t)count, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
  }
  if (!on_device) (void)::kpm::dev_free(dg, e == hipSuccess);
  if (e != hipSuccess) {
    kpm::set_error("kpm_kernel_factors: %s", hipGetErrorString(e));
    return ::kpm::hip_status(e);
  }
  return KPM_OK;
}

extern "C" int kpm_reconstruct_jackson(const double* mu, int32_t M, const double* energies_ev, int32_t K,
                                       double e_min, double e_max, double* rho, int32_t on_device,
                                       void* hip_stream) {
  kpm::clear_error();
  return kpm::reconstruct("kpm_reconstruct_jackson", kpm::kKernelJackson, mu, M, energies_ev, K, e_min, e_max, 0.0,
                          rho, nullptr, on_device, hip_stream);
}

extern "C" int kpm_reconstruct_lorentz(const double* mu, int32_t M, const double* energies_ev, int32_t K,
                                       double e_min, double e_max, double lambda, double* rho, int32_t on_device,
                                       void* hip_stream) {
  kpm::clear_error();
  if (!(std::isfinite(lambda) && lambda > 0.0)) {
    kpm::set_error("kpm_reconstruct_lorentz: need lambda > 0");
    return KPM_E_INVALID;
  }
  return kpm::reconstruct("kpm_reconstruct_lorentz", kpm::kKernelLorentz, mu, M, energies_ev, K, e_min, e_max, lambda,
                          rho, nullptr, on_device, hip_stream);
}

extern "C" int kpm_reconstruct_cpgf(const double* mu, int32_t M, const double* energies_ev, int32_t K, double e_min,
                                    double e_max, double eta_ev, double* rho, double* green, int32_t on_device,
                                    void* hip_stream) {
  kpm::clear_error();
  if (!(std::isfinite(eta_ev) && eta_ev > 0.0)) {
    kpm::set_error("kpm_reconstruct_cpgf: need eta > 0");
    return KPM_E_INVALID;
  }
  return kpm::reconstruct("kpm_reconstruct_cpgf", 2, mu, M, energies_ev, K, e_min, e_max, eta_ev, rho, green,
                          on_device, hip_stream);
}

namespace kpm {

// ---------------------------------------------------------------------------
// Kubo-Bastin and optical conductivity.
//
// Both contract Gamma with the delta function's coefficients on one side and
// the CPGF coefficients of eqs. green_function_cheb_expansion(b) on the other,
// integrated over the energy with the Fermi function f (eq. cond 1st order,
// eq. delta_function_cheb_expansion, eq. conductivity_1st_order).  With eps =
// cos(theta), Delta_n d eps = D_n d theta, D_n = (2/pi) cos(n theta); theta runs
// over Q equal cells of [0, pi]: the integrand apart from f at each cell's
// midpoint, times the cell's occupation weight int_cell f(cos theta) d theta.
//
// D is real and the same for every Fermi energy and frequency, so Gamma meets D
// first, as real matrix products over the series index n,
//     V_m(q) = sum_n D_n(q) Gamma_nm,   U_m(q) = sum_n D_n(q) Gamma_mn,
// and the complex coefficients, which depend on the broadening and frequency,
// only act on V and U, O(Q M) per frequency.  cos(n (pi - theta)) =
// (-1)^n cos(n theta) pairs cell q with Q - 1 - q: the even and odd orders are
// summed apart for q < Q/2 and give both cells, half the operations again.
// (The complex products sum_m g_m(q) Gamma_nm of a table of g with Gamma and its
// transpose, per frequency, take 16 Q M^2 operations; V and U take 4 Q M^2, the
// combination that the Bastin formula needs 2 Q M^2.)
// ---------------------------------------------------------------------------
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kLT = 64;          // tile: theta cells (of the lower half) and columns
constexpr int kLK = 16;          // series indices per LDS stage
constexpr int kLP = kLT + 16;    // LDS pitch: the two rows of half an operand read use different halves of the banks
constexpr int kFermiSub = 32;    // sub-cells per cell in the occupation weights at T > 0

// The grid: cell q has its midpoint at (q + 1/2) pi / Q; rows of the lower half
// q0 <= q < q0 + nq (nq <= Qh = ceil(Q/2)) padded to nqp, a multiple of kLT.
struct ThetaRows {
  int Q, q0, nq, nqp;
};

// D[n][i] = (2/pi) cos(n theta_q), q = q0 + i, zero for n >= M and in the
// padding; 16 orders per thread.  n (2 q + 1) pi / (2 Q) is reduced exactly
// (n (2 q + 1) mod 4 Q) before the cosine.
__global__ void theta_table_kernel(ThetaRows g, int M, double* __restrict__ D) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.nqp) return;
  const int n0 = blockIdx.y * 16;
  const uint32_t period = 4u * (uint32_t)g.Q, step = 2u * (uint32_t)(g.q0 + i) + 1u;
  uint32_t idx = (uint32_t)(((uint64_t)n0 * step) % period);
  const double inv = 1.0 / (2.0 * g.Q);
  for (int j = 0; j < 16; ++j) {
    const int n = n0 + j;
    D[(int64_t)n * g.nqp + i] = (n < M && i < g.nq) ? 2.0 / M_PI * cospi((double)idx * inv) : 0.0;
    idx += step;
    if (idx >= period) idx -= period;
  }
}

// The right operand B [Mp][C] (zero-padded rows and columns), from Gamma [M][M]:
// NCOL = 2 (Bastin): columns 2 m, 2 m + 1 = Im Gamma_nm - Im Gamma_mn, Re Gamma_nm + Re Gamma_mn;
// NCOL = 4 (optical): columns 4 m .. 4 m + 3 = Gamma_nm, Gamma_mn (re, im).
template <int NCOL>
__global__ void __launch_bounds__(256) gamma_columns_kernel(const double* __restrict__ gamma, int M, int Mp, int C,
                                                            double* __restrict__ B) {
  __shared__ double2 tr[32][33];
  const int n0 = blockIdx.y * 32, m0 = blockIdx.x * 32;
  const int x = threadIdx.x % 32, y = threadIdx.x / 32;
  // (The caller's array is aligned to its doubles only.)
  auto G = [&](int64_t i) { return make_double2(gamma[2 * i], gamma[2 * i + 1]); };
  for (int j = y; j < 32; j += 8) {
    const int m = m0 + j, n = n0 + x;
    tr[j][x] = (m < M && n < M) ? G((int64_t)m * M + n) : make_double2(0.0, 0.0);
  }
  __syncthreads();
  for (int j = y; j < 32; j += 8) {
    const int n = n0 + j, m = m0 + x;
    if (n >= Mp || NCOL * m >= C) continue;
    const double2 a = (n < M && m < M) ? G((int64_t)n * M + m) : make_double2(0.0, 0.0);
    const double2 b = tr[x][j];
    double* dst = B + (int64_t)n * C + NCOL * m;
    if constexpr (NCOL == 2) {
      dst[0] = a.y - b.y;
      dst[1] = a.x + b.x;
    } else {
      dst[0] = a.x;
      dst[1] = a.y;
      dst[2] = b.x;
      dst[3] = b.y;
    }
  }
}

// Inner root w of w^2 - 2 z w + 1 (|w| < 1 for Im z > 0).
__device__ inline cplx inner_root(cplx z) {
  const cplx r = csqrt_p({z.re * z.re - z.im * z.im - 1.0, 2.0 * z.re * z.im});
  const cplx wp = {z.re + r.re, z.im + r.im}, wm = {z.re - r.re, z.im - r.im};
  return cdiv({1.0, 0.0}, (hypot(wp.re, wp.im) >= hypot(wm.re, wm.im)) ? wp : wm);
}

// Factors of the retarded derivative g'_m = -2 i w^m (i m / s^2 + z / s^3), s =
// sqrt(1 - z^2) = i (w - z), at z = cos(theta_q) + i eta: fine[q][j] = w^j (j <
// 32), coarse[q][t] = w^(32 t), sc[q] = (1/s^2, z/s^3).
__global__ void cpgf_factors_kernel(int Q, int nt, double eta, double2* __restrict__ fine, double2* __restrict__ coarse,
                                    double2* __restrict__ sc) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= Q) return;
  const cplx z = {cospi((q + 0.5) / Q), eta};
  const cplx w = inner_root(z);
  const cplx s = {-(w.im - z.im), w.re - z.re};
  const cplx s2 = cmul(s, s);
  const cplx c1 = cdiv({1.0, 0.0}, s2), c2 = cdiv(z, cmul(s2, s));
  sc[2 * (int64_t)q] = make_double2(c1.re, c1.im);
  sc[2 * (int64_t)q + 1] = make_double2(c2.re, c2.im);
  cplx p = {1.0, 0.0};
  for (int j = 0; j < 32; ++j) {
    fine[(int64_t)q * 32 + j] = make_double2(p.re, p.im);
    p = cmul(p, w);
  }
  cplx c = {1.0, 0.0};
  for (int t = 0; t < nt; ++t) {
    coarse[(int64_t)q * nt + t] = make_double2(c.re, c.im);
    c = cmul(c, p);
  }
}

// Epilogue operands of the product D^T B.
struct SeriesOut {
  double* W = nullptr;                                        // BASTIN = false: W[2 i], W[2 i + 1] = rows q, Q - 1 - q
  const double2 *fine = nullptr, *coarse = nullptr, *sc = nullptr;   // BASTIN = true
  int nt = 0;
  double* part = nullptr;                                     // [column tile][Q]
};

// D [Mp][nqp], B [Mp][C]: the sums over the even (E) and odd (O) orders n of D B
// on a 64 x 64 tile; E + O is the row of cell q, E - O that of cell Q - 1 - q.
// Four waves of 2 x 2 FP64 MFMA tiles for E and for O.  Panels of 16 orders go
// global memory -> registers (two panels ahead) -> one of two LDS stages, in
// rows ordered even orders first, one barrier per panel.
// BASTIN: the tile's sum over its 32 orders m of Im [g'_m V_m - conj(g'_m) U_m] =
// Re g'_m (Im V_m - Im U_m) + Im g'_m (Re V_m + Re U_m); otherwise the rows of W.
//
// Bound by the FP64 matrix rate (one workgroup's 64 x 64 x 16 panel is 1024 clocks
// of MFMA per wave, its loads 16 KB).  M = 1024, Q = 4096: the complex products
// on vector FMAs took 2.0 ms (34 TFLOP/s over eight times the operations); this
// takes 0.215 ms (40 TFLOP/s, a large FP64 product reaches 71).  With its tables
// and Fermi sums the Hall curve of 64 energies went from 2.6 to 0.34 ms, the
// optical reconstruction at M = 512, 4 frequencies from 2.4 to 0.2 ms.
template <bool BASTIN>
__global__ void __launch_bounds__(256) series_gemm_kernel(const double* __restrict__ D, const double* __restrict__ B,
                                                          ThetaRows g, int Mp, int C, SeriesOut out) {
  __shared__ __attribute__((aligned(16))) double la[2][kLK][kLP], lb[2][kLK][kLP];
  const int lane = threadIdx.x & 63, r = lane & 15, q4 = lane >> 4;
  const int wave = threadIdx.x >> 6;
  const int wi = (wave & 1) * 32, wj = (wave >> 1) * 32;
  const int i0 = blockIdx.y * kLT, c0 = blockIdx.x * kLT;
  const int row = threadIdx.x / 16, col = 4 * (threadIdx.x % 16);
  const int lrow = (row & 1) * 8 + (row >> 1);
  const int chunks = Mp / kLK;
  typedef f64x2 Panel[4];
  auto load = [&](int c, Panel& p) {
    const double* pa = D + (int64_t)(c * kLK + row) * g.nqp + i0 + col;
    const double* pb = B + (int64_t)(c * kLK + row) * C + c0 + col;
    p[0] = *reinterpret_cast<const f64x2*>(pa);
    p[1] = *reinterpret_cast<const f64x2*>(pa + 2);
    p[2] = *reinterpret_cast<const f64x2*>(pb);
    p[3] = *reinterpret_cast<const f64x2*>(pb + 2);
  };
  auto store = [&](const Panel& p, int st) {
    *reinterpret_cast<f64x2*>(&la[st][lrow][col]) = p[0];
    *reinterpret_cast<f64x2*>(&la[st][lrow][col + 2]) = p[1];
    *reinterpret_cast<f64x2*>(&lb[st][lrow][col]) = p[2];
    *reinterpret_cast<f64x2*>(&lb[st][lrow][col + 2]) = p[3];
  };
  f64x4 acc[2][2][2];   // [even, odd][row tile][column tile]
#pragma unroll
  for (int par = 0; par < 2; ++par)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[par][i][j] = f64x4{};
  auto product = [&](int st) {
    double a[4][2], b[4][2];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[k][i] = la[st][4 * k + q4][wi + 16 * i + r];
        b[k][i] = lb[st][4 * k + q4][wj + 16 * i + r];
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[k >> 1][i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[k][i], b[k][j], acc[k >> 1][i][j], 0, 0, 0);
  };
  Panel p0, p1;
  load(0, p0);
  load(min(1, chunks - 1), p1);
  store(p0, 0);
  load(min(2, chunks - 1), p0);
  // Chunk c is in LDS stage c % 2, chunks c + 1 and c + 2 are on their way (past
  // the last chunk, the last one again).
  auto step = [&](int c, Panel& p, int st) {
    lds_barrier();
    store(p, st ^ 1);
    load(min(c + 3, chunks - 1), p);
    product(st);
  };
  int c = 0;
  for (; c + 2 <= chunks; c += 2) {
    step(c, p1, 0);
    step(c + 1, p0, 1);
  }
  if (c < chunks) step(c, p1, 0);
  // Element e of a tile: row 4 e + lane / 16, column lane % 16.
  if constexpr (!BASTIN) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int l = i0 + wi + 16 * i + 4 * e + q4;
          if (l >= g.nq) continue;
          const double ev = acc[0][i][j][e], od = acc[1][i][j][e];
          double* dst = out.W + (int64_t)(2 * l) * C + c0 + wj + 16 * j + r;
          dst[0] = ev + od;
          dst[C] = ev - od;
        }
  } else {
    __shared__ double red[2][2][kLT];   // [column wave][cell of the pair][row]
    const bool odd = (r & 1) != 0;      // odd columns carry the Im g' part
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int rowl = wi + 16 * i + 4 * e + q4;
        const int ql = min(g.q0 + i0 + rowl, (g.Q - 1) / 2);
#pragma unroll
        for (int side = 0; side < 2; ++side) {
          const int64_t q = side ? g.Q - 1 - ql : ql;
          const double2 cw = out.coarse[q * out.nt + blockIdx.x];
          const double2 s1 = out.sc[2 * q], s2 = out.sc[2 * q + 1];
          double sum = 0.0;
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int ml = (wj + 16 * j + r) >> 1;
            const double m = (double)(32 * (int)blockIdx.x + ml);
            const double2 fw = out.fine[q * 32 + ml];
            const cplx w = cmul({cw.x, cw.y}, {fw.x, fw.y});
            const cplx h = cmul(w, {-m * s1.y + s2.x, m * s1.x + s2.y});   // g' = -2 i h
            const double v = side ? acc[0][i][j][e] - acc[1][i][j][e] : acc[0][i][j][e] + acc[1][i][j][e];
            sum += (odd ? -2.0 * h.re : 2.0 * h.im) * v;
          }
#pragma unroll
          for (int x = 1; x < 16; x <<= 1) sum += __shfl_xor(sum, x);
          if (r == 0) red[wave >> 1][side][rowl] = sum;
        }
      }
    __syncthreads();
    if (threadIdx.x < 2 * kLT) {
      const int side = threadIdx.x / kLT, rowl = threadIdx.x % kLT;
      const int ql = g.q0 + i0 + rowl;
      if (i0 + rowl < g.nq) {
        const int q = side ? g.Q - 1 - ql : ql;
        // (The middle cell of an odd Q is its own partner and has one writer, side 0.)
        if (side == 0 || q != ql) out.part[(int64_t)blockIdx.x * g.Q + q] = red[0][side][rowl] + red[1][side][rowl];
      }
    }
  }
}

// out[q] = sum_t part[t][q].
__global__ void sum_tiles_kernel(const double* __restrict__ part, int nt, int Q, double* __restrict__ out) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= Q) return;
  double s = 0.0;
  for (int t = 0; t < nt; ++t) s += part[(int64_t)t * Q + q];
  out[q] = s;
}

// cosines of the sub-cell midpoints, [kFermiSub][Q] (T > 0).
__global__ void sub_cosine_kernel(int Q, double* __restrict__ cs) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= Q) return;
  const int j = blockIdx.y;
  cs[(int64_t)j * Q + q] = cospi((kFermiSub * (double)q + j + 0.5) / (kFermiSub * (double)Q));
}

// Occupation weight of cell q: int_cell f(cos theta) d theta, f the Fermi
// function 1/(1 + exp((eps - mu~)/kT~)) in rescaled energies.  kT~ = 0: the
// length of the cell inside [theta_mu, pi] (theta_mu = arccos mu~, 0 or pi
// outside the spectrum); kT~ > 0: midpoint sum over kFermiSub equal sub-cells.
__device__ inline double occ_weight(int q, int Q, double mut, double kTt, const double* __restrict__ cs) {
  const double h = M_PI / Q;
  const double lo = q * h;
  if (kTt == 0.0) {
    const double th_mu = (mut >= 1.0) ? 0.0 : (mut <= -1.0 ? M_PI : acos(mut));
    return fmin(fmax(lo + h - fmax(lo, th_mu), 0.0), h);
  }
  double acc = 0.0;
  for (int j = 0; j < kFermiSub; ++j) {
    const double x = (cs[(int64_t)j * Q + q] - mut) / kTt;
    const double ex = exp(-fabs(x));   // no overflow on either side of mu
    acc += (x > 0.0) ? ex / (1.0 + ex) : 1.0 / (1.0 + ex);
  }
  return acc * (h / kFermiSub);
}

// Fixed-order tree over a workgroup of 256.
__device__ inline double block_sum(double x, double* red) {
  __syncthreads();
  red[threadIdx.x] = x;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  return red[0];
}

// psum[k][s] = sum over cells 256 s .. 256 s + 255 of F_q w_q(E_k): one workgroup
// per energy and 256 cells (one per energy alone took 218 us at 64 energies, T > 0).
__global__ void bastin_sigma_kernel(const double* __restrict__ F, int Q, const double* __restrict__ energies,
                                    double e_min, double e_max, double kTt, const double* __restrict__ cs,
                                    double* __restrict__ psum) {
  __shared__ double red[256];
  const int k = blockIdx.x;
  const double de_p = 0.5 * (e_max + e_min), de_m = 0.5 * (e_max - e_min);
  const double mut = (energies[k] - de_p) / de_m;
  const int q = blockIdx.y * 256 + threadIdx.x;
  double x = 0.0;
  if (q < Q) {
    const double wq = occ_weight(q, Q, mut, kTt, cs);
    if (wq > 0.0) x = F[q] * wq;
  }
  const double s = block_sum(x, red);
  if (threadIdx.x == 0) psum[(int64_t)k * gridDim.y + blockIdx.y] = s;
}

// sigma[k] = scale * sum_s psum[k][s].
__global__ void bastin_final_kernel(const double* __restrict__ psum, int ns, double scale, double* sigma) {
  __shared__ double red[256];
  double x = 0.0;
  for (int i = threadIdx.x; i < ns; i += 256) x += psum[(int64_t)blockIdx.x * ns + i];
  const double s = block_sum(x, red);
  if (threadIdx.x == 0) sigma[blockIdx.x] = scale * s;
}

// Sizes shared by both reconstructions.
struct SeriesShape {
  int Q, Qh, Mp, C;
  SeriesShape(int M, int n_theta, int ncol) {
    Q = n_theta > 0 ? n_theta : 4 * M;
    Qh = (Q + 1) / 2;
    Mp = (int)ceil_div(M, kLK) * kLK;
    C = (int)ceil_div((int64_t)ncol * M, kLT) * kLT;
  }
};

// Pieces of one device allocation, 256-byte aligned.
struct Carve {
  size_t used = 0;
  size_t add(size_t bytes) {
    const size_t at = used;
    used += (bytes + 255) & ~(size_t)255;
    return at;
  }
};

}  // namespace kpm

extern "C" int kpm_reconstruct_sigma_bastin(const double* gamma, int32_t M, const double* energies_ev, int32_t K,
                                            double e_min, double e_max, double eta_ev, double kT_ev,
                                            double orbitals_per_nm2, int32_t n_theta, double* sigma,
                                            int32_t on_device, void* hip_stream) {
  using namespace kpm;
  clear_error();
  KPM_CHECK_ARG(gamma && energies_ev && sigma, "NULL argument");
  KPM_CHECK_ARG(M >= 1 && M <= 16384 && K >= 1, "need 1 <= M <= 16384 and K >= 1");
  KPM_CHECK_ARG(std::isfinite(e_min) && std::isfinite(e_max) && e_min < e_max, "need e_min < e_max");
  KPM_CHECK_ARG(eta_ev > 0.0 && std::isfinite(eta_ev), "eta must be > 0");
  KPM_CHECK_ARG(kT_ev >= 0.0 && std::isfinite(kT_ev), "kT must be >= 0");
  KPM_CHECK_ARG(orbitals_per_nm2 > 0.0, "orbitals_per_nm2 must be > 0");
  KPM_CHECK_ARG(n_theta >= 0 && n_theta <= (1 << 20), "n_theta must be in [0, 2^20]");
  const SeriesShape sh(M, n_theta, 2);
  const int Q = sh.Q, nt = sh.C / kLT, ns = (int)ceil_div(Q, 256);
  const ThetaRows rows = {Q, 0, sh.Qh, (int)ceil_div(sh.Qh, kLT) * kLT};
  // Energies per block: their partial sums take at most 256 MB.
  const int k_max = std::min(K, std::max(1, (1 << 25) / ns));
  hipStream_t s = (hipStream_t)hip_stream;
  const double de_m = 0.5 * (e_max - e_min);
  const size_t gn = (size_t)M * M * 2;
  Carve cv;
  const size_t o_b = cv.add(sizeof(double) * (size_t)sh.Mp * sh.C), o_d = cv.add(sizeof(double) * (size_t)sh.Mp * rows.nqp);
  const size_t o_fine = cv.add(sizeof(double2) * 32 * (size_t)Q), o_coarse = cv.add(sizeof(double2) * (size_t)Q * nt);
  const size_t o_sc = cv.add(sizeof(double2) * 2 * (size_t)Q), o_part = cv.add(sizeof(double) * (size_t)Q * nt);
  const size_t o_f = cv.add(sizeof(double) * (size_t)Q), o_ps = cv.add(sizeof(double) * (size_t)k_max * ns);
  const size_t o_cs = cv.add(kT_ev > 0.0 ? sizeof(double) * kFermiSub * (size_t)Q : 0);
  const size_t o_host = cv.add(on_device ? 0 : sizeof(double) * (gn + 2 * (size_t)K));
  char* ws = nullptr;
  KPM_TRY_HIP(::kpm::dev_malloc(&ws, cv.used));
  auto at = [&](size_t o) { return (double*)(ws + o); };
  const double* dg = gamma;
  const double* den = energies_ev;
  double* dsig = sigma;
  hipError_t e = hipSuccess;
  if (!on_device) {
    double* h = at(o_host);
    e = hipMemcpyAsync(h, gamma, sizeof(double) * gn, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(h + gn, energies_ev, sizeof(double) * K, hipMemcpyHostToDevice, s);
    dg = h;
    den = h + gn;
    dsig = h + gn + K;
  }
  if (e == hipSuccess) {
    SeriesOut out;
    out.fine = (double2*)at(o_fine);
    out.coarse = (double2*)at(o_coarse);
    out.sc = (double2*)at(o_sc);
    out.nt = nt;
    out.part = at(o_part);
    const unsigned qb = (unsigned)ceil_div(Q, 256);
    hipLaunchKernelGGL(theta_table_kernel, dim3((unsigned)ceil_div(rows.nqp, 256), sh.Mp / 16), dim3(256), 0, s, rows,
                       M, at(o_d));
    hipLaunchKernelGGL(gamma_columns_kernel<2>, dim3((unsigned)ceil_div(sh.C / 2, 32), (unsigned)ceil_div(sh.Mp, 32)),
                       dim3(256), 0, s, dg, M, sh.Mp, sh.C, at(o_b));
    hipLaunchKernelGGL(cpgf_factors_kernel, dim3((unsigned)ceil_div(Q, 64)), dim3(64), 0, s, Q, nt, eta_ev / de_m,
                       (double2*)at(o_fine), (double2*)at(o_coarse), (double2*)at(o_sc));
    hipLaunchKernelGGL(series_gemm_kernel<true>, dim3(nt, rows.nqp / kLT), dim3(256), 0, s, at(o_d), at(o_b), rows,
                       sh.Mp, sh.C, out);
    hipLaunchKernelGGL(sum_tiles_kernel, dim3((unsigned)ceil_div(Q, 64)), dim3(64), 0, s, at(o_part), nt, Q, at(o_f));
    if (kT_ev > 0.0)
      hipLaunchKernelGGL(sub_cosine_kernel, dim3(qb, kFermiSub), dim3(256), 0, s, Q, at(o_cs));
    for (int k0 = 0; k0 < K; k0 += std::min(k_max, K - k0)) {
      const int kn = std::min(k_max, K - k0);
      hipLaunchKernelGGL(bastin_sigma_kernel, dim3(kn, ns), dim3(256), 0, s, at(o_f), Q, den + k0, e_min, e_max,
                         kT_ev / de_m, at(o_cs), at(o_ps));
      // pref = -2 pi i (N/Omega)/de-^2 is imaginary: Re(pref F) = -Im(pref) Im(F).
      hipLaunchKernelGGL(bastin_final_kernel, dim3(kn), dim3(256), 0, s, at(o_ps), ns,
                         2.0 * M_PI * orbitals_per_nm2 / (de_m * de_m), dsig + k0);
    }
    e = ::kpm::launch_status();
  }
  if (e == hipSuccess && !on_device) {
    e = hipMemcpyAsync(sigma, dsig, sizeof(double) * K, hipMemcpyDeviceToHost, s);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)::kpm::dev_free(ws, e == hipSuccess);
  if (e != hipSuccess) {
    set_error("kpm_reconstruct_sigma_bastin: %s", hipGetErrorString(e));
    return ::kpm::hip_status(e);
  }
  return KPM_OK;
}

namespace kpm {

// ---------------------------------------------------------------------------
// Optical conductivity sigma_ab(omega) at chemical potential mu and
// temperature T (eq. cond 1st order, rank-1 and rank-2 Gamma of eq. Gammanm,
// Lambda_n and Lambda_nm(omega), combined as in eq. conductivity_1st_order):
//   sigma(w)/(e^2/h) = (-2 pi i (N/Omega)/E_w) [ sum_n Gamma_n L_n + (1/de-) sum_nm Gamma_nm L_nm(w) ],
//   L_n = int f Delta_n,  L_nm(w) = int f [g^R_n(eps + w~) Delta_m + Delta_n g^A_m(eps - w~)],
// i.e. per cell sum_m [g^A_m(eps - w~) V_m + g^R_m(eps + w~) U_m] with V and U as
// above, once for all frequencies.  V and U are formed for blocks of cells, so
// that the workspace stays near a gigabyte.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) occ_weights_kernel(int Q, double mut, double kTt, const double* __restrict__ cs,
                                                          double* __restrict__ w) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < Q) w[q] = occ_weight(q, Q, mut, kTt, cs);
}

// x1[q] = sum_n Gamma1_n D_n(q) (complex) for both cells of each pair: 64 pairs
// per workgroup, the orders split over its 16 waves.
__global__ void __launch_bounds__(1024) optical_rank1_kernel(const double* __restrict__ D, ThetaRows g, int M,
                                                             const double* __restrict__ g1, double2* __restrict__ x1) {
  __shared__ double red[16][64][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane;   // < nqp
  double er = 0.0, ei = 0.0, dr = 0.0, di = 0.0;
#pragma unroll 4
  for (int n = 2 * wave; n < M; n += 32) {
    const double d0 = D[(int64_t)n * g.nqp + i];
    er += d0 * g1[2 * n];
    ei += d0 * g1[2 * n + 1];
    if (n + 1 < M) {
      const double d1 = D[(int64_t)(n + 1) * g.nqp + i];
      dr += d1 * g1[2 * n + 2];
      di += d1 * g1[2 * n + 3];
    }
  }
  red[wave][lane][0] = er;
  red[wave][lane][1] = ei;
  red[wave][lane][2] = dr;
  red[wave][lane][3] = di;
  __syncthreads();
  if (wave == 0 && i < g.nq) {
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int w = 0; w < 16; ++w)
#pragma unroll
      for (int x = 0; x < 4; ++x) s[x] += red[w][lane][x];
    const int q = g.q0 + i;
    x1[q] = make_double2(s[0] + s[2], s[1] + s[3]);
    if (g.Q - 1 - q != q) x1[g.Q - 1 - q] = make_double2(s[0] - s[2], s[1] - s[3]);
  }
}

// p[k][q] = sum_m [g^A_m(eps_q - w~_k) V_m(q) + g^R_m(eps_q + w~_k) U_m(q)], g_m =
// -2 w^m / (w - z): one wave per cell and kOptK frequencies, lane l taking the
// orders l, l + 64, ... (w^l by squarings, then steps of w^64).
constexpr int kOptK = 4;
__global__ void __launch_bounds__(256) optical_para_kernel(const double* __restrict__ W, ThetaRows g, int M, int C,
                                                           const double* __restrict__ omegas, int K, double de_m,
                                                           double eta, double2* __restrict__ p) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // row of W
  if (row >= 2 * (int64_t)g.nq) return;
  const int ql = g.q0 + (int)(row >> 1);
  const int q = (row & 1) ? g.Q - 1 - ql : ql;
  if ((row & 1) && q == ql) return;   // the middle cell of an odd Q: row 0 of its pair alone
  const int k0 = blockIdx.y * kOptK;
  const double eps = cospi((q + 0.5) / g.Q);
  cplx pw[kOptK][2], st[kOptK][2], sum[kOptK][2], pre[kOptK][2];   // [frequency][retarded at +w, advanced at -w]
#pragma unroll
  for (int k = 0; k < kOptK; ++k)
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const double wt = omegas[min(k0 + k, K - 1)] / de_m;
      const cplx z = {eps + (a ? -wt : wt), eta};
      const cplx w = inner_root(z);
      pre[k][a] = cdiv({-2.0, 0.0}, {w.re - z.re, w.im - z.im});
      cplx b = w, x = {1.0, 0.0};
#pragma unroll
      for (int bit = 0; bit < 6; ++bit) {
        if ((lane >> bit) & 1) x = cmul(x, b);
        b = cmul(b, b);
      }
      pw[k][a] = x;
      st[k][a] = b;
      sum[k][a] = {0.0, 0.0};
    }
  const double2* wr = reinterpret_cast<const double2*>(W + row * C);
  for (int m = lane; m < M; m += 64) {
    const double2 v = wr[2 * m], u = wr[2 * m + 1];
#pragma unroll
    for (int k = 0; k < kOptK; ++k) {
      // Retarded: w^m U_m;  advanced: conj(w^m) V_m.
      const cplx x = pw[k][0], y = pw[k][1];
      sum[k][0].re += x.re * u.x - x.im * u.y;
      sum[k][0].im += x.re * u.y + x.im * u.x;
      sum[k][1].re += y.re * v.x + y.im * v.y;
      sum[k][1].im += y.re * v.y - y.im * v.x;
      pw[k][0] = cmul(x, st[k][0]);
      pw[k][1] = cmul(y, st[k][1]);
    }
  }
#pragma unroll
  for (int k = 0; k < kOptK; ++k) {
    const cplx r = cmul(pre[k][0], sum[k][0]);
    const cplx a = cmul({pre[k][1].re, -pre[k][1].im}, sum[k][1]);
    double re = r.re + a.re, im = r.im + a.im;
#pragma unroll
    for (int x = 1; x < 64; x <<= 1) {
      re += __shfl_xor(re, x);
      im += __shfl_xor(im, x);
    }
    if (lane == 0 && k0 + k < K) p[(int64_t)(k0 + k) * g.Q + q] = make_double2(re, im);
  }
}

// sigma[k] = -2 pi i (N/Omega)/E_k sum_q w_q (x1_q + p_kq / de-), stored (re, im).
__global__ void __launch_bounds__(256) optical_final_kernel(const double2* __restrict__ x1, const double2* __restrict__ p,
                                                            const double* __restrict__ w, int Q,
                                                            const double* __restrict__ omegas, double de_m, double opn,
                                                            double* sigma) {
  __shared__ double red[256];
  const int k = blockIdx.x;
  double l[2] = {0.0, 0.0}, a[2] = {0.0, 0.0};
  for (int q = threadIdx.x; q < Q; q += 256) {
    const double wq = w[q];
    if (wq <= 0.0) continue;
    const double2 x = x1[q], y = p[(int64_t)k * Q + q];
    l[0] += wq * x.x;
    l[1] += wq * x.y;
    a[0] += wq * y.x;
    a[1] += wq * y.y;
  }
  const double lr = block_sum(l[0], red), li = block_sum(l[1], red);
  const double ar = block_sum(a[0], red), ai = block_sum(a[1], red);
  if (threadIdx.x == 0) {
    const double xr = lr + ar / de_m, xi = li + ai / de_m;
    const double c = 2.0 * M_PI * opn / omegas[k];
    sigma[2 * k] = c * xi;        // -i (xr + i xi) = xi - i xr
    sigma[2 * k + 1] = -c * xr;
  }
}

}  // namespace kpm

extern "C" int kpm_reconstruct_sigma_optical(const double* gamma_nm, const double* gamma_n, int32_t M,
                                             const double* omegas_ev, int32_t K, double mu_ev, double e_min,
                                             double e_max, double eta_ev, double kT_ev, double orbitals_per_nm2,
                                             int32_t n_theta, double* sigma, int32_t on_device, void* hip_stream) {
  using namespace kpm;
  clear_error();
  KPM_CHECK_ARG(gamma_nm && gamma_n && omegas_ev && sigma, "NULL argument");
  KPM_CHECK_ARG(M >= 1 && M <= 16384 && K >= 1 && K <= 65536, "need 1 <= M <= 16384 and 1 <= K <= 65536");
  KPM_CHECK_ARG(std::isfinite(e_min) && std::isfinite(e_max) && e_min < e_max, "need e_min < e_max");
  KPM_CHECK_ARG(std::isfinite(mu_ev), "mu must be finite");
  KPM_CHECK_ARG(eta_ev > 0.0 && std::isfinite(eta_ev), "eta must be > 0");
  KPM_CHECK_ARG(kT_ev >= 0.0 && std::isfinite(kT_ev), "kT must be >= 0");
  KPM_CHECK_ARG(orbitals_per_nm2 > 0.0, "orbitals_per_nm2 must be > 0");
  KPM_CHECK_ARG(n_theta >= 0 && n_theta <= (1 << 20), "n_theta must be in [0, 2^20]");
  hipStream_t s = (hipStream_t)hip_stream;
  // The frequencies are checked on the host.
  std::vector<double> om;
  try {
    om.resize((size_t)K);
  } catch (...) {
    set_error("kpm_reconstruct_sigma_optical: out of host memory");
    return KPM_E_NOMEM;
  }
  if (on_device) {
    KPM_TRY_HIP(hipMemcpyAsync(om.data(), omegas_ev, sizeof(double) * K, hipMemcpyDeviceToHost, s));
    KPM_TRY_SYNC(hipStreamSynchronize(s));
  } else {
    std::memcpy(om.data(), omegas_ev, sizeof(double) * K);
  }
  for (double w : om) KPM_CHECK_ARG(w > 0.0 && std::isfinite(w), "every frequency must be > 0 (hbar omega in eV)");
  const SeriesShape sh(M, n_theta, 4);
  const int Q = sh.Q;
  const double de_p = 0.5 * (e_max + e_min), de_m = 0.5 * (e_max - e_min);
  const double mut = (mu_ev - de_p) / de_m;
  const double kTt = kT_ev / de_m;
  // Pairs of cells per block: V and U of a block take at most about 1 GB.
  const int64_t cap = ((int64_t)1 << 30) / (2 * (int64_t)sizeof(double) * sh.C) / kLT * kLT;
  const int nq_max = (int)std::min<int64_t>(ceil_div(sh.Qh, kLT) * kLT, std::max<int64_t>(kLT, cap));
  // Frequencies per block: their sums per cell take at most about 1 GB.  V and U are
  // formed again for each block of frequencies only where they come in several blocks.
  const int k_max = (int)std::min<int64_t>(
      K, std::max<int64_t>(kOptK, ((int64_t)1 << 30) / ((int64_t)sizeof(double2) * Q) / kOptK * kOptK));
  const size_t gn = (size_t)M * M * 2;
  Carve cv;
  const size_t o_b = cv.add(sizeof(double) * (size_t)sh.Mp * sh.C), o_d = cv.add(sizeof(double) * (size_t)sh.Mp * nq_max);
  const size_t o_w = cv.add(2 * sizeof(double) * (size_t)nq_max * sh.C), o_p = cv.add(sizeof(double2) * (size_t)k_max * Q);
  const size_t o_x1 = cv.add(sizeof(double2) * (size_t)Q), o_occ = cv.add(sizeof(double) * (size_t)Q);
  const size_t o_cs = cv.add(kT_ev > 0.0 ? sizeof(double) * kFermiSub * (size_t)Q : 0);
  const size_t o_host = cv.add(on_device ? 0 : sizeof(double) * (gn + 2 * (size_t)M + 3 * (size_t)K));
  char* ws = nullptr;
  KPM_TRY_HIP(::kpm::dev_malloc(&ws, cv.used));
  auto at = [&](size_t o) { return (double*)(ws + o); };
  const double* dgnm = gamma_nm;
  const double* dgn = gamma_n;
  const double* dom = omegas_ev;
  double* dsig = sigma;
  hipError_t e = hipSuccess;
  if (!on_device) {
    double* h = at(o_host);
    e = hipMemcpyAsync(h, gamma_nm, sizeof(double) * gn, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(h + gn, gamma_n, sizeof(double) * 2 * M, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(h + gn + 2 * M, omegas_ev, sizeof(double) * K, hipMemcpyHostToDevice, s);
    dgnm = h;
    dgn = h + gn;
    dom = h + gn + 2 * M;
    dsig = h + gn + 2 * M + K;
  }
  if (e == hipSuccess) {
    const unsigned qb = (unsigned)ceil_div(Q, 256);
    hipLaunchKernelGGL(gamma_columns_kernel<4>, dim3((unsigned)ceil_div(sh.C / 4, 32), (unsigned)ceil_div(sh.Mp, 32)),
                       dim3(256), 0, s, dgnm, M, sh.Mp, sh.C, at(o_b));
    if (kT_ev > 0.0)
      hipLaunchKernelGGL(sub_cosine_kernel, dim3(qb, kFermiSub), dim3(256), 0, s, Q, at(o_cs));
    hipLaunchKernelGGL(occ_weights_kernel, dim3(qb), dim3(256), 0, s, Q, mut, kTt, at(o_cs), at(o_occ));
    for (int k0 = 0; k0 < K && e == hipSuccess; k0 += k_max) {   // (K <= 65536)
      const int kn = std::min(k_max, K - k0);
      for (int q0 = 0; q0 < sh.Qh && e == hipSuccess; q0 += nq_max) {
        ThetaRows rows = {Q, q0, std::min(nq_max, sh.Qh - q0), 0};
        rows.nqp = (int)ceil_div(rows.nq, kLT) * kLT;
        if (k0 == 0 || sh.Qh > nq_max) {
          SeriesOut out;
          out.W = at(o_w);
          hipLaunchKernelGGL(theta_table_kernel, dim3((unsigned)ceil_div(rows.nqp, 256), sh.Mp / 16), dim3(256), 0, s,
                             rows, M, at(o_d));
          hipLaunchKernelGGL(optical_rank1_kernel, dim3(rows.nqp / 64), dim3(1024), 0, s, at(o_d), rows, M, dgn,
                             (double2*)at(o_x1));
          hipLaunchKernelGGL(series_gemm_kernel<false>, dim3(sh.C / kLT, rows.nqp / kLT), dim3(256), 0, s, at(o_d),
                             at(o_b), rows, sh.Mp, sh.C, out);
        }
        hipLaunchKernelGGL(optical_para_kernel,
                           dim3((unsigned)ceil_div(2 * (int64_t)rows.nq, 4), (unsigned)ceil_div(kn, kOptK)), dim3(256), 0,
                           s, at(o_w), rows, M, sh.C, dom + k0, kn, de_m, eta_ev / de_m, (double2*)at(o_p));
        e = ::kpm::launch_status();
      }
      if (e == hipSuccess) {
        hipLaunchKernelGGL(optical_final_kernel, dim3(kn), dim3(256), 0, s, (double2*)at(o_x1), (double2*)at(o_p),
                           at(o_occ), Q, dom + k0, de_m, orbitals_per_nm2, dsig + 2 * (size_t)k0);
        e = ::kpm::launch_status();
      }
    }
  }
  if (e == hipSuccess && !on_device) e = hipMemcpyAsync(sigma, dsig, sizeof(double) * 2 * K, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)::kpm::dev_free(ws, e == hipSuccess);
  if (e != hipSuccess) {
    set_error("kpm_reconstruct_sigma_optical: %s", hipGetErrorString(e));
    return ::kpm::hip_status(e);
  }
  return KPM_OK;
}
