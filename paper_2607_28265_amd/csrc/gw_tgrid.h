// Index maps and register passes of the time-grid transform (gw_tgrid.hip),
// host and device: L = D1 D2 16 points, an in-place decimation-in-frequency
// FFT in three passes.
//   pass 1, lane r < L / D1: DFT over x[r + (L / D1) q], q < D1, output k1
//           times exp(-2 pi i r k1 / L), stored at r + (L / D1) k1;
//   pass 2, lane n3 + 16 k1 (n3 < 16, k1 < D1): DFT over the D2 values at
//           n3 + 16 q + (L / D1) k1, output k2 times exp(-2 pi i n3 k2 / (16 D2)),
//           stored in place;
//   pass 3, lane g < L / 16: DFT over the 16 values at 16 g + n3; output k3 is
//           X[tg_owned(L, D1, D2, g, k3)].
#pragma once

#include <math.h>

#include <vector>

#include "gw_fft.h"
#include "gw_tgplan.h"

namespace gw {

constexpr int kTgMaxL = 4096;

// LDS position of element i: one pad element per 16.
__host__ __device__ inline int tg_pad(int i) { return i + (i >> 4); }

// The transform index that lane `lane` (< L / 16) holds in output slot k3 of
// the last pass: k1 + D1 k2 + (L / 16) k3 with k1 = lane / D2, k2 = lane mod D2.
__host__ __device__ inline int tg_owned(int L, int D1, int D2, int lane, int k3) {
  return lane / D2 + D1 * (lane % D2) + (L / 16) * k3;
}

// Pass radices for a length L = 2^q, 16 <= L <= 4096.
inline bool tgrid_plan(int L, int* D1, int* D2) {
  if (L < 16 || L > kTgMaxL || (L & (L - 1)) != 0) return false;
  if (L >= 256) {
    *D1 = L / 256;
    *D2 = 16;
  } else {
    *D1 = 1;
    *D2 = L / 16;
  }
  return true;
}

// First pass on one lane's D1 inputs (only v[0 .. NZ) may be nonzero, the
// rest hold zero), w = exp(-2 pi i r / L); outputs in natural order.
template <int D1, int NZ>
__host__ __device__ inline void tg_pass1(double2* v, double2 w) {
  if constexpr (D1 > 1) {
    if constexpr (D1 == 16) {
      Dft<16>::template run_slots_nz<NZ>(v);
    } else {
      Dft<D1>::run_slots(v);
    }
    double2 o[D1];
#pragma unroll
    for (int k = 0; k < D1; ++k) o[k] = v[dft_slot<D1>(k)];
    double2 t = w;
#pragma unroll
    for (int k = 1; k < D1; ++k) {
      o[k] = c_mul(o[k], t);
      if (k + 1 < D1) t = c_mul(t, w);
    }
#pragma unroll
    for (int k = 0; k < D1; ++k) v[k] = o[k];
  }
}

// Second pass on one lane's D2 values, w = exp(-2 pi i n3 / (16 D2)).
template <int D2>
__host__ __device__ inline void tg_pass2(double2* v, double2 w) {
  if constexpr (D2 > 1) {
    Dft<D2>::run_slots(v);
    double2 o[D2];
#pragma unroll
    for (int k = 0; k < D2; ++k) o[k] = v[dft_slot<D2>(k)];
    double2 t = w;
#pragma unroll
    for (int k = 1; k < D2; ++k) {
      o[k] = c_mul(o[k], t);
      if (k + 1 < D2) t = c_mul(t, w);
    }
#pragma unroll
    for (int k = 0; k < D2; ++k) v[k] = o[k];
  }
}

// exp(-i pi k / 16), k = 0 .. 15
__host__ __device__ inline double2 w32(int k) {
  constexpr double c[9] = {1.0,                 0.98078528040323044, 0.92387953251128674, 0.83146961230254524,
                           0.70710678118654752, 0.55557023301960222, 0.38268343236508977, 0.19509032201612827, 0.0};
  return k <= 8 ? make_double2(c[k], -c[8 - k]) : make_double2(-c[16 - k], -c[k - 8]);
}

// Kaiser-Bessel gridding (Beatty, Nishimura & Pauly 2005): a sample at grid
// coordinate x is spread over kTgW grid points (gw_tgplan.h) with weights
// psi(x - g) = I0(beta sqrt(1 - (2 (x - g) / kTgW)^2)) / I0(beta),
// whose transform sum_g psi(x - g) exp(-2 pi i g nu) is
// psi_hat(nu) exp(-2 pi i x nu) up to the images at nu + 1, nu - 1, ...
constexpr int kTgLead = kTgW / 2 - 1;  // grid points before the sample's cell

// I0(x), 0 <= x <= 44, by its power series (85 terms: the rest below 1e-30).
struct TgBessel {
  double c[85];
  TgBessel() {
    c[0] = 1.0;
    for (int k = 1; k < 85; ++k) c[k] = c[k - 1] / ((double)k * (double)k);
  }
  double operator()(double x) const {
    const double q = 0.25 * x * x;
    double s = c[84];
    for (int k = 83; k >= 0; --k) s = s * q + c[k];
    return s;
  }
};

// Shape for |nu| <= nu_max: close to the largest beta that keeps the images
// at |nu| >= 1 - nu_max beyond the main lobe, 2 % below it (measured error
// over all nu and x: 7e-15 of sum |y| at nu_max 1/8, 5e-14 at 1/5 (the default
// window), 6e-13 at 1/4; 0.96 and 1.0 of it 7e-13 and 2e-12 there).
inline double tgrid_beta(double nu_max) { return 0.98 * 3.141592653589793 * kTgW * (1.0 - nu_max); }

inline double tgrid_psi_hat(double nu, double beta, double i0_beta) {
  const double x = 3.141592653589793 * kTgW * nu, a = sqrt(beta * beta - x * x);
  return kTgW * sinh(a) / (a * i0_beta);
}

// The kTgW weights of a sample at offset s of its cell (0 <= s < 1): grid
// point m of the window is s + kTgLead - m away.
// I0(beta sqrt(1 - u^2)) is analytic in u, so each weight is a Chebyshev series
// in s (26 terms: the rest below 1e-17), a tenth of the work of its Bessel
// series.
struct TgWindow {
  static constexpr int kTerms = 26;
  double c[kTerms][kTgW];

  explicit TgWindow(double beta) {
    const TgBessel i0;
    const double i0_beta = i0(beta);
    double v[kTerms][kTgW];
    for (int j = 0; j < kTerms; ++j)
      for (int m = 0; m < kTgW; ++m) {
        const double u = 2.0 / kTgW * (0.5 + 0.5 * cos(angle(1, j)) + kTgLead - m);
        v[j][m] = i0(beta * sqrt(1.0 - u * u)) / i0_beta;
      }
    for (int k = 0; k < kTerms; ++k) {
      for (int m = 0; m < kTgW; ++m) c[k][m] = 0.0;
      for (int j = 0; j < kTerms; ++j) {
        const double t = (k == 0 ? 1.0 : 2.0) / kTerms * cos(angle(k, j));
        for (int m = 0; m < kTgW; ++m) c[k][m] += t * v[j][m];
      }
    }
  }
  static double angle(int k, int j) { return 3.141592653589793 * k * (j + 0.5) / kTerms; }
  void weights(double s, double* w) const {
    const double t = 2.0 * s - 1.0;
    double p[kTgW] = {}, q[kTgW] = {};
    for (int k = kTerms - 1; k > 0; --k)
      for (int m = 0; m < kTgW; ++m) {
        const double n = c[k][m] + 2.0 * t * p[m] - q[m];
        q[m] = p[m];
        p[m] = n;
      }
    for (int m = 0; m < kTgW; ++m) w[m] = c[0][m] + t * p[m] - q[m];
  }
};

}  // namespace gw
