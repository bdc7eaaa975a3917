// GW+C tail: the numerical Landau cumulant on the time grid, the cumulant
// propagator, the FFT to frequency and the spectral function.
//
//   c_j   = q_j |Im Sigma_j| / (pi nu_j^2),  nu_j = w_j - eps_n   (c_j = 0 at nu_j = 0)
//   C~(t) = sum_j c_j (e^{-i nu_j t} - 1)                  (Eq. landau_cumulant_truncated)
//   G(t)  = -i theta(t) e^{-i E_QP t - eta t} e^{C~(t)}    (Eq. cumulant_propagator_numerical_time)
//   G(w_l) = dt sum_k G(t_k) e^{i w_l t_k}                 (Eqs. cumulant_propagator_fourier,
//                                                          cumulant_propagator_convolution)
//   A(w)  = -Im G(w) / pi                                  (Eq. eq:AGWC)
//
// With w_l = w_0 + l d_omega and dt = 2 pi / (n_t d_omega) the sum over k is an
// inverse DFT of G(t_k) e^{i w_0 t_k}; the factor e^{i w_0 t_k} and dt are
// folded into the time-domain kernel.  The n_t x n_real complex exponentials
// are products of tabulated ones; the FFT is a Stockham of radix 16, whose last
// pass writes the spectral function.
#include <utility>

#include "gwc_internal.h"

namespace gwc {

constexpr double PI_D = 3.14159265358979323846;

// One block: trapezoid weights, nu_j, c_j, and (Z, 1 - Z).
__global__ void __launch_bounds__(256)
cumulant_weights_kernel(const double *__restrict__ w, const double *__restrict__ im, int n_real,
                        double eps_n, double *__restrict__ nu, double *__restrict__ c,
                        double *__restrict__ z_out) {
  __shared__ double sh[256];
  const int tid = threadIdx.x;
  double acc = 0.0;
  for (int j = tid; j < n_real; j += 256) {
    double q = 0.0;
    if (n_real > 1) {
      if (j > 0) q += 0.5 * (w[j] - w[j - 1]);
      if (j < n_real - 1) q += 0.5 * (w[j + 1] - w[j]);
    }
    const double v = w[j] - eps_n;
    const double g = fabs(im[j]) / PI_D;
    const double cj = (v != 0.0) ? q * g / (v * v) : 0.0;
    nu[j] = v;
    c[j] = cj;
    acc += cj;
  }
  sh[tid] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) sh[tid] += sh[tid + s];
    __syncthreads();
  }
  if (tid == 0 && z_out) {
    const double Z = exp(-sh[0]);
    z_out[0] = Z;
    z_out[1] = 1.0 - Z;
  }
}

void launch_cumulant_weights(const double *omega_real, const double *im_sigma, int n_real,
                             double eps_n, double *nu, double *c, double *z_out,
                             hipStream_t stream) {
  cumulant_weights_kernel<<<1, 256, 0, stream>>>(omega_real, im_sigma, n_real, eps_n, nu, c,
                                                 z_out);
}

// C~(t) and G(t) for 256 NA time points a workgroup.  With k = k0 + 256 a + 64 d
// + b (a < NA, d < 4, b a lane),
//   e^{-i nu_j t_k} = e^{-i nu_j (k0 + 256 a) dt} e^{-i nu_j b dt} e^{-i nu_j 64 d dt},
// the middle factor a product of 8 and 8 tabulated ones and the last a power, so
// that a frequency needs NA + 17 sines and cosines a workgroup and a time point
// five multiply-adds; one sincos each (about 400 cycles a wave) before: 269 -> 54 us
// at n_t = 2^18, n_real = 400.  The tables' phases nu t are formed without
// rounding the product: the phase error of a point is no larger than one
// rounded product's (2.4e-13 rms against 3.4e-13 there).  The four waves take
// every fourth frequency and their sums are added in order at the end.
constexpr int CT_J = 64;  // frequencies at a time

__device__ __forceinline__ double2 phase_factor(double nu, double t) {
  const double x = nu * t, lo = fma(nu, t, -x);
  double s, c;
  sincos(x, &s, &c);
  return make_double2(fma(-s, lo, c), -fma(c, lo, s));
}

template <int NA>
__global__ void __launch_bounds__(256)
cumulant_time_kernel(const double *__restrict__ nu, const double *__restrict__ c, int n_real,
                     int n_t, double dt, double e_qp, double omega0, double eta,
                     double2 *__restrict__ Gt) {
  constexpr int Q = NA + 17;
  // per frequency: c_j e^{-i nu_j (k0 + 256 a) dt}; b dt, b < 8; 8 b dt; 64 dt.
  // At the end the waves' sums.
  __shared__ double2 T[CT_J * Q > 4 * 4 * NA * 64 ? CT_J * Q : 4 * 4 * NA * 64];
  __shared__ double csum[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int k0 = blockIdx.x * (256 * NA);
  double cr[4][NA], ci[4][NA], total = 0.0;
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      cr[d][a] = 0.0;
      ci[d][a] = 0.0;
    }
  for (int j0 = 0; j0 < n_real; j0 += CT_J) {
    const int nj = min(CT_J, n_real - j0);
    __syncthreads();
    for (int e = tid; e < nj * Q; e += 256) {
      const int j = e / Q, q = e - j * Q;
      const int k = q < NA ? k0 + 256 * q : (q < NA + 8 ? q - NA : (q < NA + 16 ? 8 * (q - NA - 8) : 64));
      double2 x = phase_factor(nu[j0 + j], (double)k * dt);
      if (q < NA) {
        const double w = c[j0 + j];
        x = make_double2(w * x.x, w * x.y);
      }
      T[e] = x;
    }
    __syncthreads();
#pragma unroll 2
    for (int j = wave; j < nj; j += 4) {
      const double2 *Tj = T + j * Q;
      const double2 p = Tj[NA + (lane & 7)], q = Tj[NA + 8 + (lane >> 3)], g = Tj[NA + 16];
      double2 y = make_double2(p.x * q.x - p.y * q.y, p.x * q.y + p.y * q.x);
      total += c[j0 + j];
#pragma unroll
      for (int d = 0; d < 4; ++d) {
#pragma unroll
        for (int a = 0; a < NA; ++a) {
          const double2 x = Tj[a];
          cr[d][a] = fma(-x.y, y.y, fma(x.x, y.x, cr[d][a]));
          ci[d][a] = fma(x.y, y.x, fma(x.x, y.y, ci[d][a]));
        }
        if (d < 3) y = make_double2(y.x * g.x - y.y * g.y, y.x * g.y + y.y * g.x);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int a = 0; a < NA; ++a) T[((wave * NA + a) * 4 + d) * 64 + lane] = make_double2(cr[d][a], ci[d][a]);
  if (lane == 0) csum[wave] = total;
  __syncthreads();
  const double cs = (csum[0] + csum[1]) + (csum[2] + csum[3]);
#pragma unroll
  for (int a = 0; a < NA; ++a) {
    const int i = a * 256 + tid, k = k0 + i;
    if (k >= n_t) continue;
    const double2 s0 = T[i], s1 = T[NA * 256 + i], s2 = T[2 * NA * 256 + i], s3 = T[3 * NA * 256 + i];
    const double sr = (s0.x + s1.x) + (s2.x + s3.x), si = (s0.y + s1.y) + (s2.y + s3.y);
    const double t = (double)k * dt;
    const double theta = (k == 0) ? 0.5 : 1.0;
    const double mag = theta * dt * exp((sr - cs) - eta * t);
    const double phi = si - (e_qp - omega0) * t;
    double s, co;
    sincos(phi, &s, &co);
    // -i * mag * (cos phi + i sin phi)
    Gt[k] = make_double2(mag * s, -mag * co);
  }
}

void launch_cumulant_time(const double *nu, const double *c, int n_real, int n_t, double dt,
                          double e_qp, double omega0, double eta, double2 *Gt,
                          hipStream_t stream) {
  // 1024 points a workgroup where that still gives every CU one
  if (n_t >= 1 << 18)
    cumulant_time_kernel<4><<<n_t / 1024, 256, 0, stream>>>(nu, c, n_real, n_t, dt, e_qp, omega0, eta, Gt);
  else
    cumulant_time_kernel<1><<<(n_t + 255) / 256, 256, 0, stream>>>(nu, c, n_real, n_t, dt, e_qp, omega0, eta, Gt);
}

// y_p = sum_q x_q e^{2 pi i p q / R} in registers, R a power of two up to 16.
template <int R>
__device__ __forceinline__ void small_dft(double (&re)[R], double (&im)[R]) {
  constexpr double C[8] = {1.0, 0.92387953251128675613, 0.70710678118654752440, 0.38268343236508977173,
                           0.0, -0.38268343236508977173, -0.70710678118654752440, -0.92387953251128675613};
  constexpr double S[8] = {0.0, 0.38268343236508977173, 0.70710678118654752440, 0.92387953251128675613,
                           1.0, 0.92387953251128675613, 0.70710678118654752440, 0.38268343236508977173};
  constexpr int L = R == 2 ? 1 : R == 4 ? 2 : R == 8 ? 3 : 4;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    int r = 0;
#pragma unroll
    for (int b = 0; b < L; ++b) r |= ((i >> b) & 1) << (L - 1 - b);
    if (r > i) {
      const double x = re[i], y = im[i];
      re[i] = re[r];
      im[i] = im[r];
      re[r] = x;
      im[r] = y;
    }
  }
#pragma unroll
  for (int len = 2; len <= R; len *= 2)
#pragma unroll
    for (int i = 0; i < R; i += len)
#pragma unroll
      for (int k = 0; k < len / 2; ++k) {
        const double wc = C[k * (16 / len)], ws = S[k * (16 / len)];
        const double x = re[i + k + len / 2], y = im[i + k + len / 2];
        const double vr = k == 0 ? x : x * wc - y * ws, vi = k == 0 ? y : x * ws + y * wc;
        const double ur = re[i + k], ui = im[i + k];
        re[i + k] = ur + vr;
        im[i + k] = ui + vi;
        re[i + k + len / 2] = ur - vr;
        im[i + k + len / 2] = ui - vi;
      }
}

// One Stockham pass of radix R of the unnormalised inverse DFT (e^{+2 pi i l k / n}):
// the m-point transforms of the passes before become m R-point ones.  A pass is
// bound by its launch and one round trip to memory (5 us): 18 passes of radix 2
// at n = 2^18 took 87 us, these five 26 us.  LAST:
// only A[l] = -Im / pi of the first n_out results is written.
template <int R, bool LAST>
__global__ void __launch_bounds__(64)
fft_pass_kernel(const double2 *__restrict__ in, double2 *__restrict__ out, int nr, int m, double *__restrict__ A,
                int n_out) {
  const int j = blockIdx.x * 64 + threadIdx.x;
  if (j >= nr) return;
  const int k = j & (m - 1);
  double re[R], im[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const double2 x = in[j + (long long)q * nr];
    re[q] = x.x;
    im[q] = x.y;
  }
  if (m > 1) {
    const double step = 2.0 / ((double)m * R) * (double)k;  // exact: m R is a power of two
#pragma unroll
    for (int q = 1; q < R; ++q) {
      double s, c;
      sincospi(step * q, &s, &c);
      const double x = re[q], y = im[q];
      re[q] = x * c - y * s;
      im[q] = x * s + y * c;
    }
  }
  small_dft<R>(re, im);
  const int o = (j - k) * R + k;
#pragma unroll
  for (int p = 0; p < R; ++p) {
    const int l = o + p * m;
    if (LAST) {
      if (l < n_out) A[l] = -im[p] / PI_D;
    } else {
      out[l] = make_double2(re[p], im[p]);
    }
  }
}

void launch_fft_spectrum(double2 *buf_a, double2 *buf_b, int log2n, int n_out, double *A_out, hipStream_t stream) {
  const int n = 1 << log2n;
  double2 *in = buf_a, *out = buf_b;
  int m = 1;
  auto pass = [&](int bits) {
    const int nr = n >> bits, grid = (nr + 63) / 64;
    switch (bits) {
      case 1: fft_pass_kernel<2, false><<<grid, 64, 0, stream>>>(in, out, nr, m, nullptr, 0); break;
      case 2: fft_pass_kernel<4, false><<<grid, 64, 0, stream>>>(in, out, nr, m, nullptr, 0); break;
      case 3: fft_pass_kernel<8, false><<<grid, 64, 0, stream>>>(in, out, nr, m, nullptr, 0); break;
      default:
        if (m == nr) fft_pass_kernel<16, true><<<grid, 64, 0, stream>>>(in, out, nr, m, A_out, n_out);
        else fft_pass_kernel<16, false><<<grid, 64, 0, stream>>>(in, out, nr, m, nullptr, 0);
    }
    m <<= bits;
    std::swap(in, out);
  };
  if (log2n % 4) pass(log2n % 4);
  for (int b = 0; b < log2n / 4; ++b) pass(4);
}

}  // namespace gwc
