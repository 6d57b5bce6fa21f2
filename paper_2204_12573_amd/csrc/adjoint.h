// Adjoint (force) terms of the paper's Section V.B reordering, shared by the standalone
// adjoint kernel and the fused descriptor / quadratic-form / adjoint kernel.
//
// With g_i = de_i/dd~_i and d~_{(a,b),l} = sum_m c_a c_b:
//   u_{a,l,m} = de_i/dc_{a,l,m} = sum_b G^_{ab,l} c_{b,l,m},
//               G^_{ab,l} = g_{(min,max),l}, doubled on the diagonal a = b.
// For each listed pair p = (i, j, s) inside the cutoff, with Delta = r_j + s L - r_i:
//   w_p = de_i/dDelta = sum_{n,l,m} u_{(s_j,n),l,m} grad_Delta [R_n(r) Y_lm(Delta/r)]
//       = u^ sum_n (R_n' Z_n - R_n Zl_n / r) + (1/r) sum_lm A_lm grad P_lm(u^)
//   with Z_n = sum_lm u_{n,lm} Y_lm, Zl_n = sum_lm l u_{n,lm} Y_lm, A_lm = sum_n u_{n,lm} R_n,
// and w_p = 0 outside the cutoff.
#pragma once

#include "basis.h"
#include "half.h"
#include "pair.h"

namespace flare {

// sum_lm A_lm grad P_lm(x, y, z)
__device__ __forceinline__ void poly_grad_dot(const float* A, float x, float y, float z,
                                              float& gx, float& gy, float& gz) {
#pragma clang fp contract(off)
  const float xx = x * x, yy = y * y, zz = z * z;
  const float xy = x * y, xz = x * z, yz = y * z, dxy = xx - yy, z4 = 4.f * zz;
  gx = kY1 * A[3];
  gx = fmaf(kY2a * y, A[4], gx);
  gx = fmaf(kY2a * z, A[7], gx);
  gx = fmaf(-2.f * kY20 * x, A[6], gx);
  gx = fmaf(2.f * kY22 * x, A[8], gx);
  gx = fmaf(6.f * kY33 * xy, A[9], gx);
  gx = fmaf(kY32a * yz, A[10], gx);
  gx = fmaf(-2.f * kY31 * xy, A[11], gx);
  gx = fmaf(-6.f * kY30 * xz, A[12], gx);
  gx = fmaf(kY31 * (fmaf(-3.f, xx, z4) - yy), A[13], gx);
  gx = fmaf(2.f * kY32b * xz, A[14], gx);
  gx = fmaf(3.f * kY33 * dxy, A[15], gx);
  gy = kY1 * A[1];
  gy = fmaf(kY2a * x, A[4], gy);
  gy = fmaf(kY2a * z, A[5], gy);
  gy = fmaf(-2.f * kY20 * y, A[6], gy);
  gy = fmaf(-2.f * kY22 * y, A[8], gy);
  gy = fmaf(3.f * kY33 * dxy, A[9], gy);
  gy = fmaf(kY32a * xz, A[10], gy);
  gy = fmaf(kY31 * (fmaf(-3.f, yy, z4) - xx), A[11], gy);
  gy = fmaf(-6.f * kY30 * yz, A[12], gy);
  gy = fmaf(-2.f * kY31 * xy, A[13], gy);
  gy = fmaf(-2.f * kY32b * yz, A[14], gy);
  gy = fmaf(-6.f * kY33 * xy, A[15], gy);
  gz = kY1 * A[2];
  gz = fmaf(kY2a * y, A[5], gz);
  gz = fmaf(kY2a * x, A[7], gz);
  gz = fmaf(4.f * kY20 * z, A[6], gz);
  gz = fmaf(kY32a * xy, A[10], gz);
  gz = fmaf(8.f * kY31 * yz, A[11], gz);
  gz = fmaf(kY30 * fmaf(-3.f, xx + yy, 6.f * zz), A[12], gz);
  gz = fmaf(8.f * kY31 * xz, A[13], gz);
  gz = fmaf(kY32b * dxy, A[14], gz);
}

// w = de_i/dDelta for one pair from the adjoint densities u[n][lm] of the neighbour's
// species (all 16 (l, m) in one thread).
// The radial sums are taken per (l, m): A_lm = sum_n u_{n,lm} R_n and B_lm = sum_n
// u_{n,lm} R_n', so that sum_n (R_n' Z_n - R_n Zl_n / r) = sum_lm Y_lm (B_lm - (l/r) A_lm).
template <class U>
__device__ __forceinline__ void pair_force(const PairGeom& pg, float rc, U u, float& wx, float& wy,
                                           float& wz) {
#pragma clang fp contract(off)
  float R[NR], dR[NR], Y[NLM];
  radial_d(pg.r, rc, R, dR);
  sph_harm(pg.ux, pg.uy, pg.uz, Y);
  float A[NLM], B[NLM];
#pragma unroll
  for (int lm = 0; lm < NLM; ++lm) {
    A[lm] = 0.f;
    B[lm] = 0.f;
  }
#pragma unroll
  for (int n = 0; n < NR; ++n)
#pragma unroll
    for (int lm = 0; lm < NLM; ++lm) {
      const float un = u(n, lm);
      A[lm] = fmaf(un, R[n], A[lm]);
      B[lm] = fmaf(un, dR[n], B[lm]);
    }
  const float inv_r = __builtin_amdgcn_rcpf(pg.r);   // 1 ulp; r >= the shortest pair distance
  const float il[LMAX + 1] = {0.f, inv_r, 2.f * inv_r, 3.f * inv_r};
  float s1 = 0.f;
#pragma unroll
  for (int lm = 0; lm < NLM; ++lm) s1 = fmaf(Y[lm], fmaf(-il[lm_l(lm)], A[lm], B[lm]), s1);
  float gx, gy, gz;
  poly_grad_dot(A, pg.ux, pg.uy, pg.uz, gx, gy, gz);
  wx = fmaf(pg.ux, s1, gx * inv_r);
  wy = fmaf(pg.uy, s1, gy * inv_r);
  wz = fmaf(pg.uz, s1, gz * inv_r);
}

__device__ __forceinline__ int pair_index_same(int na, int nb) {
  // packed index of (na <= nb) inside a single-species block, row-major
  return na * NR - na * (na - 1) / 2 + (nb - na);
}

// Two lanes per row (see half.h): c[n][q] holds the densities of (l, m) = 8h + q of the
// row's single neighbour species. In place, c becomes u = G^ c, group by group: lane h's
// q fall in three groups of constant l, {0}, {1,2,3}, {4..7}, with l = (0,1,2) for h = 0
// and (2,3,3) for h = 1. g(k) = g of packed component k = 4*(radial pair) + l, read as
// g[k * gstride].
__device__ __forceinline__ void u_transform_half(const float* g, int gstride, int h, float (&c)[NR][NQ]) {
  const int lg0 = h ? 2 : 0, lg1 = h ? 3 : 1, lg2 = h ? 3 : 2;
#pragma unroll
  for (int grp = 0; grp < 3; ++grp) {
    const int l = grp == 0 ? lg0 : (grp == 1 ? lg1 : lg2);
    const int q0 = grp == 0 ? 0 : (grp == 1 ? 1 : 4);
    const int q1 = grp == 0 ? 1 : (grp == 1 ? 4 : 8);
    float gh[NR][NR];
#pragma unroll
    for (int na = 0; na < NR; ++na)
#pragma unroll
      for (int nb = na; nb < NR; ++nb) {
        const float val = g[(size_t)(pair_index_same(na, nb) * 4 + l) * gstride];
        gh[na][nb] = na == nb ? 2.f * val : val;
        gh[nb][na] = gh[na][nb];
      }
#pragma unroll
    for (int q = q0; q < q1; ++q) {
      float col[NR];
#pragma unroll
      for (int n = 0; n < NR; ++n) col[n] = c[n][q];
#pragma unroll
      for (int n = 0; n < NR; ++n) {
        float acc = 0.f;
#pragma unroll
        for (int m = 0; m < NR; ++m) acc = fmaf(gh[n][m], col[m], acc);
        c[n][q] = acc;
      }
    }
  }
}

// Exchange the two halves of u so that both lanes of the row hold all of it, then split
// the row's slots between the lanes (k = h, h + 2, ...): each pair term is evaluated once
// and scattered to the reverse pair's slot of w_in, where the force gather of the
// neighbour reads it; the row's own terms are summed (each lane over its slots in order,
// then the two lanes) into f_own[R].
__device__ __forceinline__ void adjoint_pairs_half(const SlotView& v, int R, int h, const float (&c)[NR][NQ],
                                                   float4* __restrict__ f_own) {
  float u[NR][NLM];
#pragma unroll
  for (int n = 0; n < NR; ++n)
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const float other = xor1(c[n][q]);
      u[n][q] = h ? other : c[n][q];
      u[n][NQ + q] = h ? c[n][q] : other;
    }
  const int S = wave_slice(R);
  const int base = v.slice_base[S];
  const int len = v.slice_base[S + 1] - base;
  const size_t s0 = (size_t)base * 32 + (R & 31);
  float sx = 0.f, sy = 0.f, sz = 0.f;
  // lane h takes slots k = h, h + 2, ...: the geometry and reverse index of its next two
  // slots are in flight while two are evaluated, in two register groups that take turns
  // (unconditional loads, past the slice re-reading its last slot)
  auto load = [&](int k, float4& g, int& r) {
    const size_t sl = s0 + (size_t)min(k, len - 1) * 32;
    g = v.geom[sl];
    r = v.rev[sl];
  };
  auto term = [&](int k, const float4& gk, int rk) {
    if (k >= len) return;
    PairGeom pg;
    int sp;
    float wx = 0.f, wy = 0.f, wz = 0.f;
    if (unpack_geom(gk, pg, sp)) pair_force(pg, v.rc, [&](int n, int lm) { return u[n][lm]; }, wx, wy, wz);
    v.w_in[rk] = make_float4(wx, wy, wz, 0.f);
    sx += wx;
    sy += wy;
    sz += wz;
  };
  if (len > 0) {
    float4 ga[2], gb[2];
    int ra[2], rb[2];
    load(h, ga[0], ra[0]);
    load(h + 2, ga[1], ra[1]);
    for (int k0 = h; k0 < len; k0 += 8) {
      load(k0 + 4, gb[0], rb[0]);
      load(k0 + 6, gb[1], rb[1]);
      term(k0, ga[0], ra[0]);
      term(k0 + 2, ga[1], ra[1]);
      load(k0 + 8, ga[0], ra[0]);
      load(k0 + 10, ga[1], ra[1]);
      term(k0 + 4, gb[0], rb[0]);
      term(k0 + 6, gb[1], rb[1]);
    }
  }
  sx += xor1(sx);
  sy += xor1(sy);
  sz += xor1(sz);
  if (h == 0) f_own[R] = make_float4(sx, sy, sz, 0.f);
}

// The same with the row's slots split over eight lanes of four waves, for few rows: u of the 32
// rows in LDS (row stride US), each wave w of the work-group takes the slots k = h + 2 w, + 8,
// ... of its lane's row; the terms also go to LDS, where the first wave then adds the row's own
// in the order above. len <= ADJ_FEW_SLOTS.
constexpr int US = NR * NLM + 4;
constexpr int ADJ_FEW_SLOTS = 48;
__device__ __forceinline__ void adjoint_pairs_few(const SlotView& v, int R, int rl, int h, int wave,
                                                  const float* __restrict__ us, float* __restrict__ ws) {
  const int S = wave_slice(R);
  const int base = v.slice_base[S];
  const int len = v.slice_base[S + 1] - base;
  const size_t s0 = (size_t)base * 32 + (R & 31);
  const int k0 = h + 2 * wave;
  float4 g = k0 < len ? v.geom[s0 + (size_t)k0 * 32] : make_float4(0.f, 0.f, 0.f, 0.f);
  int r = k0 < len ? v.rev[s0 + (size_t)k0 * 32] : 0;
  float u[NR][NLM];
  const float4* u4 = reinterpret_cast<const float4*>(us + rl * US);
#pragma unroll
  for (int n = 0; n < NR; ++n)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 t = u4[n * 4 + q];
      u[n][4 * q] = t.x;
      u[n][4 * q + 1] = t.y;
      u[n][4 * q + 2] = t.z;
      u[n][4 * q + 3] = t.w;
    }
  for (int k = k0; k < len; k += 8) {
    const float4 gk = g;
    const int rk = r;
    const size_t next = s0 + (size_t)min(k + 8, len - 1) * 32;
    g = v.geom[next];
    r = v.rev[next];
    PairGeom pg;
    int sp;
    float wx = 0.f, wy = 0.f, wz = 0.f;
    if (unpack_geom(gk, pg, sp)) pair_force(pg, v.rc, [&](int n, int lm) { return u[n][lm]; }, wx, wy, wz);
    v.w_in[rk] = make_float4(wx, wy, wz, 0.f);
    float* w3 = ws + (k * 32 + rl) * 3;
    w3[0] = wx;
    w3[1] = wy;
    w3[2] = wz;
  }
}
__device__ __forceinline__ void adjoint_own_few(const SlotView& v, int R, int rl, int h, const float* __restrict__ ws,
                                                float4* __restrict__ f_own) {
  const int S = wave_slice(R);
  const int len = v.slice_base[S + 1] - v.slice_base[S];
  float sx = 0.f, sy = 0.f, sz = 0.f;
  for (int k = h; k < len; k += 2) {
    const float* w3 = ws + (k * 32 + rl) * 3;
    sx += w3[0];
    sy += w3[1];
    sz += w3[2];
  }
  sx += xor1(sx);
  sy += xor1(sy);
  sz += xor1(sz);
  if (h == 0) f_own[R] = make_float4(sx, sy, sz, 0.f);
}

}  // namespace flare
