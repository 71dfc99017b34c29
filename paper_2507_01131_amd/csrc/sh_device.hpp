// Real spherical harmonics of a unit vector, evaluated in registers.
//
// Basis: index l*l + l + m; real, no Condon-Shortley phase, z polar axis;
// m > 0 from Re((x+iy)^m), m < 0 from Im((x+iy)^|m|); Y_00 = 1 and
// sum_m Y_lm^2 = 2l+1.  Y_lm(u) = c_lm * P_l^m(z) * {Re,Im}(x+iy)^|m| with
// P_l^m the m-th derivative of the Legendre polynomial, generated by the
// three-term recurrence
//   (l-m+1) P_{l+1}^m = (2l+1) z P_l^m - (l+m) r^2 P_{l-1}^m,
//   P_m^m = (2m-1)!!,  P_{m+1}^m = (2m+1) z P_m^m,
// written homogeneously (r^2 kept as a variable) so that the same recurrence
// differentiated gives the gradient of the solid harmonic, from which
//   dY/dr = (grad S(u) - l S(u) u) / |r|.
// c_lm = sqrt(2l+1) sqrt((2 - [m=0]) (l-m)! / (l+m)!).
#pragma once

#include "common.hpp"

namespace tdn {

constexpr int kMaxL = 6;

constexpr double c_sqrt(double x) {
  double r = x > 1.0 ? x : 1.0;
  for (int i = 0; i < 80; ++i) r = 0.5 * (r + x / r);
  return r;
}
constexpr double c_fact(int n) { return n <= 1 ? 1.0 : n * c_fact(n - 1); }

struct ShNorm {
  float v[kMaxL + 1][kMaxL + 1];
};
constexpr ShNorm make_sh_norm() {
  ShNorm t{};
  for (int l = 0; l <= kMaxL; ++l)
    for (int m = 0; m <= l; ++m)
      t.v[l][m] = float(c_sqrt(2.0 * l + 1.0) * c_sqrt((m == 0 ? 1.0 : 2.0) * c_fact(l - m) / c_fact(l + m)));
  return t;
}
constexpr ShNorm kShNorm = make_sh_norm();

// Y(u) for a unit vector u = (x, y, z); writes (L+1)^2 values to Y[stride*i].
__device__ inline void sh_unit(int L, float x, float y, float z, float* Y, int stride = 1) {
  float re = 1.f, im = 0.f;  // (x + i y)^m
  for (int m = 0; m <= L; ++m) {
    float pmm = 1.f;
    for (int k = 1; k <= m; ++k) pmm *= float(2 * k - 1);
    float p_prev = 0.f, p = pmm;
    for (int l = m; l <= L; ++l) {
      const float c = kShNorm.v[l][m] * p;
      Y[stride * (l * l + l + m)] = c * re;
      if (m > 0) Y[stride * (l * l + l - m)] = c * im;
      // P_{l+1}^m from P_l^m and P_{l-1}^m (r^2 = 1 on the sphere)
      const float pn = (float(2 * l + 1) * z * p - float(l + m) * p_prev) / float(l - m + 1);
      p_prev = p;
      p = pn;
    }
    const float re2 = re * x - im * y;
    im = re * y + im * x;
    re = re2;
  }
}

// Y(u) for a unit vector u, all (L+1)^2 values, with L known at compile
// time: every loop unrolls, so the normalisation constants and the
// recurrence's reciprocals 1/(l - m + 1) become immediates (no table loads,
// no divisions).
template <int L>
__device__ __forceinline__ void sh_unit_all(float x, float y, float z, float* Y) {
  float re = 1.f, im = 0.f;  // (x + i y)^m
#pragma unroll
  for (int m = 0; m <= L; ++m) {
    float pmm = 1.f;
#pragma unroll
    for (int k = 1; k <= m; ++k) pmm *= float(2 * k - 1);
    float p_prev = 0.f, p = pmm;
#pragma unroll
    for (int l = m; l <= L; ++l) {
      const float c = kShNorm.v[l][m] * p;
      Y[l * l + l + m] = c * re;
      if (m > 0) Y[l * l + l - m] = c * im;
      const float pn = (float(2 * l + 1) * z * p - float(l + m) * p_prev) * (1.0f / float(l - m + 1));
      p_prev = p;
      p = pn;
    }
    const float re2 = re * x - im * y;
    im = re * y + im * x;
    re = re2;
  }
}

// Y(u) and dY/dr for r = |r| u: the direction Jacobian, [(L+1)^2][3] at
// J[stride*(3*i + a)].  Forward-mode differentiation of the recurrence with
// (value, d/dx, d/dy, d/dz) carried for every quantity.
struct Dual4 {
  float v, x, y, z;
};
__device__ __forceinline__ Dual4 dmul(Dual4 a, Dual4 b) {
  return {a.v * b.v, a.v * b.x + a.x * b.v, a.v * b.y + a.y * b.v, a.v * b.z + a.z * b.v};
}
__device__ __forceinline__ Dual4 dlin(float s, Dual4 a, float t, Dual4 b) {
  return {s * a.v + t * b.v, s * a.x + t * b.x, s * a.y + t * b.y, s * a.z + t * b.z};
}

__device__ inline void sh_unit_jacobian(int L, float x, float y, float z, float inv_norm, float* Y, float* J,
                                        int stride = 1) {
  const Dual4 X{x, 1.f, 0.f, 0.f}, Yv{y, 0.f, 1.f, 0.f}, Z{z, 0.f, 0.f, 1.f};
  const Dual4 R2{x * x + y * y + z * z, 2.f * x, 2.f * y, 2.f * z};
  Dual4 re{1.f, 0.f, 0.f, 0.f}, im{0.f, 0.f, 0.f, 0.f};
  for (int m = 0; m <= L; ++m) {
    float pmm = 1.f;
    for (int k = 1; k <= m; ++k) pmm *= float(2 * k - 1);
    Dual4 p_prev{0.f, 0.f, 0.f, 0.f}, p{pmm, 0.f, 0.f, 0.f};
    for (int l = m; l <= L; ++l) {
      const float c = kShNorm.v[l][m];
      for (int s = 0; s < (m > 0 ? 2 : 1); ++s) {
        const Dual4 S = dmul(p, s == 0 ? re : im);
        const int idx = l * l + l + (s == 0 ? m : -m);
        // S is the solid harmonic / c; Y = c S(u); dY/dr = c (grad S - l S u) / |r|
        Y[stride * idx] = c * S.v;
        const float lS = float(l) * S.v;
        J[stride * (3 * idx + 0)] = c * (S.x - lS * x) * inv_norm;
        J[stride * (3 * idx + 1)] = c * (S.y - lS * y) * inv_norm;
        J[stride * (3 * idx + 2)] = c * (S.z - lS * z) * inv_norm;
      }
      const Dual4 zp = dmul(Z, p);
      const Dual4 rp = dmul(R2, p_prev);
      const float inv = 1.f / float(l - m + 1);
      const Dual4 pn = dlin(float(2 * l + 1) * inv, zp, -float(l + m) * inv, rp);
      p_prev = p;
      p = pn;
    }
    const Dual4 re2 = dlin(1.f, dmul(re, X), -1.f, dmul(im, Yv));
    im = dlin(1.f, dmul(re, Yv), 1.f, dmul(im, X));
    re = re2;
  }
}

// The order +-m column of Y(u) and of its direction Jacobian (see
// sh_unit_jacobian), for l = m..L.
__device__ inline void sh_unit_jacobian_column(int L, int m, float x, float y, float z, float inv_norm, float* Y,
                                               float* J) {
  const Dual4 X{x, 1.f, 0.f, 0.f}, Yv{y, 0.f, 1.f, 0.f}, Z{z, 0.f, 0.f, 1.f};
  const Dual4 R2{x * x + y * y + z * z, 2.f * x, 2.f * y, 2.f * z};
  Dual4 re{1.f, 0.f, 0.f, 0.f}, im{0.f, 0.f, 0.f, 0.f};
  for (int k = 0; k < m; ++k) {
    const Dual4 re2 = dlin(1.f, dmul(re, X), -1.f, dmul(im, Yv));
    im = dlin(1.f, dmul(re, Yv), 1.f, dmul(im, X));
    re = re2;
  }
  float pmm = 1.f;
  for (int k = 1; k <= m; ++k) pmm *= float(2 * k - 1);
  Dual4 p_prev{0.f, 0.f, 0.f, 0.f}, p{pmm, 0.f, 0.f, 0.f};
  for (int l = m; l <= L; ++l) {
    const float c = kShNorm.v[l][m];
    for (int s = 0; s < (m > 0 ? 2 : 1); ++s) {
      const Dual4 S = dmul(p, s == 0 ? re : im);
      const int idx = l * l + l + (s == 0 ? m : -m);
      Y[idx] = c * S.v;
      const float lS = float(l) * S.v;
      J[3 * idx + 0] = c * (S.x - lS * x) * inv_norm;
      J[3 * idx + 1] = c * (S.y - lS * y) * inv_norm;
      J[3 * idx + 2] = c * (S.z - lS * z) * inv_norm;
    }
    const Dual4 zp = dmul(Z, p);
    const Dual4 rp = dmul(R2, p_prev);
    const float inv = 1.f / float(l - m + 1);
    const Dual4 pn = dlin(float(2 * l + 1) * inv, zp, -float(l + m) * inv, rp);
    p_prev = p;
    p = pn;
  }
}

// Gaussian radial basis: phi_q = exp(-(rn - mu_q)^2 / (2 sigma^2)),
// mu_q = q * sigma, sigma = r_cut / (n - 1); dphi_q/drn = -(rn - mu_q)/sigma^2 phi_q.
// mu_q is not rounded by itself, whatever the compiler fuses: hoisted out of a
// loop over edges its rounding alone is 2e-6 of phi_q at (rn - mu_q) = 3.5 sigma.
__device__ __forceinline__ float radial_t(float rn, int q, float sigma) { return fmaf(-float(q), sigma, rn) / sigma; }
__device__ __forceinline__ float radial_phi(float rn, int q, float sigma) {
  const float t = radial_t(rn, q, sigma);
  return expf(-0.5f * t * t);
}

}  // namespace tdn
