// Plan-time device kernels, all arithmetic in FP64:
//   * the response templates H_z(q) (Section 1: the predicted, normalised
//     Fourier response used in eq. 2),
//   * the Fourier-domain bank T_z[k] = conj(FFT_L(h_z))[k] / L with
//     h_z[q mod L] = H_z(q) (the per-segment filter of overlap-and-save,
//     Section 2), written in the hot kernel's slot order,
//   * the twiddle table W_L^j = exp(-i 2 pi j / L) of eq. 3.
//
// Template: G_z(q) = int_{-1/2}^{1/2} exp(i pi (z s^2 - 2 q s)) ds and
// H_z(q) = exp(-i pi q) G_z(q). For z > 0, completing the square,
//   G_z(q) = exp(-i pi q^2/z) / sqrt(2z) * [F(t2) - F(t1)],
//   t1 = sqrt(2z)(-1/2 - q/z), t2 = sqrt(2z)(1/2 - q/z),
// with F(x) = C(x) + i S(x) the Fresnel integrals (kernel exp(i pi t^2/2)).
// For x >= 0 write F(x) = (1+i)/2 - a(x) exp(i pi x^2/2); F is odd. Since
// (pi/2) t2^2 = pi (z/4 - q + q^2/z) and (pi/2) t1^2 = pi (z/4 + q + q^2/z),
// exp(-i pi q^2/z) exp(i pi t_{1,2}^2/2) = exp(i pi (z/4 +/- q)) exactly, so
// the only large phase left, exp(-i pi q^2/z), is reduced exactly as
// fmod(q^2, 2z)/z; it appears only when t1 < 0 < t2.
//
// a(x): for small x from the power series
//   F(x) = sum_n (i pi/2)^n x^(2n+1) / (n! (2n+1)),  a = ((1+i)/2 - F) e^{-i pi x^2/2};
// otherwise from F(x) = (1+i)/2 erf(w), w = (sqrt(pi)/2)(1 - i) x, so that
//   a(x) = (1+i)/2 * exp(w^2) erfc(w),
// with exp(w^2) erfc(w) from its Laplace continued fraction
//   sqrt(pi) exp(w^2) erfc(w) = 1/(w + (1/2)/(w + (2/2)/(w + (3/2)/(w + ...))))
// (valid for Re w > 0), evaluated from its innermost term outwards. Its error
// after N terms falls as exp(-2 Re(w) sqrt(2 N)) with Re(w) = (sqrt(pi)/2) x, so
// N = 230 / x^2 + 8 leaves it under 2e-16 from x = 1.8 on (checked in extended
// precision against 6000 terms); a fixed N makes a step one reciprocal and
// four multiply-adds. (The modified Lentz method, with its two complex
// divisions and two magnitudes per step and a test for the end, took 105 us
// for 101 x 257 values, a chain that no occupancy hides, against 12 us.)
#include <hip/hip_runtime.h>

#include <cmath>

#include "bank_sum.hpp"
#include "fft_radix.hpp"
#include "layout.hpp"

namespace fdas {

struct c64 {
  double x, y;
};

__device__ inline c64 zmul(c64 a, c64 b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ inline c64 zsub(c64 a, c64 b) { return {a.x - b.x, a.y - b.y}; }
__device__ inline c64 zscale(c64 a, double s) { return {a.x * s, a.y * s}; }
// exp(i pi u) for a real u (argument given in half-turns).
__device__ inline c64 expipi(double u) {
  double s, c;
  sincospi(u, &s, &c);
  return {c, s};
}

constexpr double kSmallX = 1.8;

// (-1)^(n/2) / (n! (2n+1)), the coefficients of the power series
constexpr double fresnel_coef(int n) {
  double f = 1.0;
  for (int i = 2; i <= n; ++i) f *= (double)i;
  return ((n / 2) & 1 ? -1.0 : 1.0) / (f * (double)(2 * n + 1));
}

// a(x) for x >= 0 (see the file comment).
__device__ c64 fresnel_aux(double x) {
  const double kPi = 3.14159265358979323846;
  if (x < kSmallX) {
    // C(x) and S(x) as polynomials in u^2, u = pi x^2 / 2 <= 5.09 (terms up to
    // u^40 / 40!, under 1e-19)
    const double u = 0.5 * kPi * x * x, u2 = u * u;
    double c = 0.0, sn = 0.0;
#pragma unroll
    for (int n = 40; n >= 0; n -= 2) c = __builtin_fma(c, u2, fresnel_coef(n));
#pragma unroll
    for (int n = 39; n >= 1; n -= 2) sn = __builtin_fma(sn, u2, fresnel_coef(n));
    const c64 e = expipi(-0.5 * x * x);
    return zmul({0.5 - c * x, 0.5 - sn * u * x}, e);
  }
  const double sp = 0.88622692545275801365;  // sqrt(pi)/2
  const double w = sp * x;  // the argument is w (1 - i)
  const int n0 = (int)(230.0 / (x * x)) + 8;
  // f = w (1 - i) + (n/2) / f, n = n0 .. 1; 1/f = conj(f) / |f|^2, with the
  // reciprocal of |f|^2 by two Newton steps from the hardware's estimate
  double fr = w, fi = -w;
  double an = 0.5 * n0;
  for (int n = n0; n > 0; --n) {
    const double d = __builtin_fma(fr, fr, fi * fi);
    double r = __builtin_amdgcn_rcp(d);
    r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
    r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
    const double t = an * r;
    fr = __builtin_fma(t, fr, w);
    fi = __builtin_fma(-t, fi, -w);
    an -= 0.5;
  }
  const double inv_sqrt_pi = 0.56418958354775628695;
  const double d = 1.0 / __builtin_fma(fr, fr, fi * fi);
  return zmul({0.5, 0.5}, {fr * d * inv_sqrt_pi, -fi * d * inv_sqrt_pi});
}

// G_z(q) for z > 0.
__device__ c64 response_g_pos(double z, double q) {
  const double rt = sqrt(2.0 * z);
  const double t1 = rt * (-0.5 - q / z);
  const double t2 = rt * (0.5 - q / z);
  const c64 p2 = expipi(fmod(0.25 * z - q, 2.0));  // e^{-i pi q^2/z} e^{i pi t2^2/2}
  const c64 p1 = expipi(fmod(0.25 * z + q, 2.0));  // e^{-i pi q^2/z} e^{i pi t1^2/2}
  const c64 a2 = zmul(fresnel_aux(fabs(t2)), p2);
  const c64 a1 = zmul(fresnel_aux(fabs(t1)), p1);
  c64 g;
  if (t1 < 0.0 && t2 >= 0.0) {
    // F(t2) - F(t1) = (1+i) - a(t2) E(t2) - a(|t1|) E(t1)
    const c64 p0 = expipi(-fmod(q * q, 2.0 * z) / z);
    g = zsub(zsub(zmul({1.0, 1.0}, p0), a2), a1);
  } else if (t1 >= 0.0) {
    // both arguments >= 0: the (1+i)/2 terms cancel exactly
    g = zsub(a1, a2);
  } else {
    // both < 0: F(t) = -(1+i)/2 + a(|t|) E(t)
    g = zsub(a2, a1);
  }
  return zscale(g, 1.0 / rt);
}

__device__ c64 template_h(double z, double q) {
  c64 g;
  if (z == 0.0) {
    const double s = (q == 0.0) ? 1.0 : sinpi(q) / (3.14159265358979323846 * q);
    g = {s, 0.0};
  } else {
    g = response_g_pos(fabs(z), q);
    if (z < 0.0) g.y = -g.y;
  }
  return zmul(expipi(-fmod(q, 2.0)), g);
}

// H[i][j] = H_{z_i}(j - m/2), z_i = -zmax + i dz. With interbin the rows
// come in pairs: H[2i][j] = H_{z_i}(j - m/2) and H[2i+1][j] = H_{z_i}(j - m/2
// - 1/2), the response at r + 1/2 from the same bins.
__global__ void templates_kernel(c64 *__restrict__ out, int rows, int m, double zmax, double dz,
                                 int interbin) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const int taps = m + 1;
  if (idx >= rows * taps) return;
  const int row = idx / taps, j = idx % taps;
  const int i = interbin ? row >> 1 : row;
  const double shift = (interbin && (row & 1)) ? 0.5 : 0.0;
  const double z = -zmax + i * dz;
  out[idx] = template_h(z, (double)(j - m / 2) - shift);
}

// W_L^j = exp(-i 2 pi j / L), rounded to FP32.
__global__ void twiddle_kernel(c32 *__restrict__ tw, int L) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= L) return;
  double s, c;
  sincospi(-2.0 * (double)j / (double)L, &s, &c);
  tw[j] = {(float)c, (float)s};
}

// bank[i][e][t] = conj(S_i(k)) / L with k the frequency of slot (t, e).
struct PutSlots {
  c32 *bank;
  LayoutDesc lay;
  __device__ void operator()(int row, int k, double re, double im) const {
    const double inv = 1.0 / (double)lay.L;
    bank[(long)row * lay.L + layout_freq_slot(lay, k)] = {(float)(re * inv), (float)(-im * inv)};
  }
};

// Natural-order copy of a slot-ordered bank: dst[i][k(t,e)] = bank[i][e][t].
__global__ void bank_natural_kernel(c32 *__restrict__ dst, const c32 *__restrict__ bank, int nz,
                                    LayoutDesc lay) {
  const int L = lay.L;
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)nz * L) return;
  const int i = (int)(idx / L);
  const int slot = (int)(idx % L);
  const int e = slot / lay.T, t = slot % lay.T;
  const int k = layout_slot_freq(lay, t, e);
  dst[(long)i * L + k] = bank[idx];
}

hipError_t launch_templates(void *out, int rows, int m, double zmax, double dz, int interbin,
                            hipStream_t s) {
  const int n = rows * (m + 1);
  hipLaunchKernelGGL(templates_kernel, dim3((n + 255) / 256), dim3(256), 0, s,
                     static_cast<c64 *>(out), rows, m, zmax, dz, interbin);
  return hipGetLastError();
}

hipError_t launch_twiddles(c32 *tw, int L, hipStream_t s) {
  hipLaunchKernelGGL(twiddle_kernel, dim3((L + 255) / 256), dim3(256), 0, s, tw, L);
  return hipGetLastError();
}

hipError_t launch_bank(c32 *bank, const void *h, int rows, int interbin, int m,
                       const LayoutDesc &lay, hipStream_t s) {
  return launch_bank_sum(h, rows, interbin, m, lay.L, PutSlots{bank, lay}, s);
}

hipError_t launch_bank_natural(c32 *dst, const c32 *bank, int nz, const LayoutDesc &lay,
                               hipStream_t s) {
  const long n = (long)nz * lay.L;
  hipLaunchKernelGGL(bank_natural_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     dst, bank, nz, lay);
  return hipGetLastError();
}

}  // namespace fdas
