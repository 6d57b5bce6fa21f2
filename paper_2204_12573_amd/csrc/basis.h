// Pair basis on the device: Chebyshev radial functions x smooth cutoff x real
// spherical harmonics, and their gradients (paper, Section V.B: B2 descriptors from
// radial functions and spherical harmonics).
//
//   R_n(r)  = T_n(x) f_c(r),  x = 2r/r_c - 1,  f_c = (r_c - r)^2 for r < r_c
//   R_n'(r) = n U_{n-1}(x) (2/r_c) f_c - 2 T_n(x) (r_c - r)
//   Y_lm(u) = P_lm(u) for a unit vector u, with P_lm the degree-l homogeneous
//             (solid harmonic) polynomial normalised so that the Y_lm are orthonormal
//   grad_Delta Y_lm(Delta/r) = (grad P_lm(u) - l P_lm(u) u) / r   (Euler's identity
//             u . grad P = l P for a homogeneous polynomial)
//
// These functions, and the others that several kernels share (half.h, adjoint.h, mixed.h and
// the epilogue of fused.hip), spell out every fused multiply-add and let the compiler form no
// others: which products of a sum it fuses depends on what surrounds the inlined code, and a
// row must give the same bits in the kernel for few rows and in the one for many.
#pragma once

#include "common.h"

namespace flare {

// normalisation constants of the real spherical harmonics, l <= 3
constexpr float kY0 = 0.28209479177387814f;    // 1/(2 sqrt(pi))
constexpr float kY1 = 0.48860251190291992f;    // sqrt(3/(4 pi))
constexpr float kY2a = 1.0925484305920792f;    // (1/2) sqrt(15/pi)
constexpr float kY20 = 0.31539156525252005f;   // (1/4) sqrt(5/pi)
constexpr float kY22 = 0.54627421529603959f;   // (1/4) sqrt(15/pi)
constexpr float kY33 = 0.59004358992664352f;   // (1/4) sqrt(35/(2 pi))
constexpr float kY32a = 2.8906114426405538f;   // (1/2) sqrt(105/pi)
constexpr float kY31 = 0.45704579946446572f;   // (1/4) sqrt(21/(2 pi))
constexpr float kY30 = 0.37317633259011540f;   // (1/4) sqrt(7/pi)
constexpr float kY32b = 1.4453057213202769f;   // (1/4) sqrt(105/pi)

__device__ __forceinline__ void sph_harm(float x, float y, float z, float* Y) {
#pragma clang fp contract(off)
  const float xx = x * x, yy = y * y, zz = z * z;
  const float dxy = xx - yy, sxy = xx + yy;
  const float xy = x * y;
  const float z4 = fmaf(4.f, zz, -sxy);        // 4 z^2 - x^2 - y^2
  Y[0] = kY0;
  Y[1] = kY1 * y;
  Y[2] = kY1 * z;
  Y[3] = kY1 * x;
  Y[4] = kY2a * xy;
  Y[5] = kY2a * (y * z);
  Y[6] = kY20 * fmaf(2.f, zz, -sxy);
  Y[7] = kY2a * (x * z);
  Y[8] = kY22 * dxy;
  Y[9] = kY33 * (y * fmaf(3.f, xx, -yy));
  Y[10] = kY32a * (xy * z);
  Y[11] = kY31 * (y * z4);
  Y[12] = kY30 * (z * fmaf(-3.f, sxy, 2.f * zz));
  Y[13] = kY31 * (x * z4);
  Y[14] = kY32b * (z * dxy);
  Y[15] = kY33 * (x * fmaf(-3.f, yy, xx));
}

__device__ __forceinline__ int lm_l(int lm) { return lm == 0 ? 0 : (lm < 4 ? 1 : (lm < 9 ? 2 : 3)); }

// R_n(r), n = 0..NR-1. x = r (2/r_c) - 1: the factor 2/r_c is loop-invariant for the
// callers, which evaluate it once.
__device__ __forceinline__ void radial(float r, float rc, float* R) {
#pragma clang fp contract(off)
  const float x = fmaf(r, 2.f / rc, -1.f);
  const float fc = (rc - r) * (rc - r);
  float t0 = 1.f, t1 = x;
  R[0] = fc;
  R[1] = x * fc;
#pragma unroll
  for (int n = 2; n < NR; ++n) {
    const float t2 = fmaf(2.f * x, t1, -t0);
    R[n] = t2 * fc;
    t0 = t1;
    t1 = t2;
  }
}

// R_n(r) and dR_n/dr = T_n'(x) (2/r_c) f_c + T_n(x) f_c', with T_n' = n U_{n-1}
__device__ __forceinline__ void radial_d(float r, float rc, float* R, float* dR) {
#pragma clang fp contract(off)
  const float dxdr = 2.f / rc;
  const float x = fmaf(r, dxdr, -1.f);
  const float q = rc - r;
  const float fc = q * q;
  const float dfc = -2.f * q;
  const float cf = dxdr * fc;
  float T[NR], U[NR];
  T[0] = 1.f;
  T[1] = x;
  U[0] = 1.f;
  U[1] = 2.f * x;
#pragma unroll
  for (int n = 2; n < NR; ++n) {
    T[n] = fmaf(2.f * x, T[n - 1], -T[n - 2]);
    U[n] = fmaf(2.f * x, U[n - 1], -U[n - 2]);
  }
  R[0] = fc;
  dR[0] = dfc;
#pragma unroll
  for (int n = 1; n < NR; ++n) {
    R[n] = T[n] * fc;
    dR[n] = fmaf((float)n * cf, U[n - 1], T[n] * dfc);
  }
}

}  // namespace flare
