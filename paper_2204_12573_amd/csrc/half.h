// Two lanes per descriptor row: lane h = 0 owns (l, m) indices 0..7 (l = 0, 1 and the
// first four m of l = 2), lane h = 1 owns 8..15 (the last m of l = 2 and l = 3). Both
// lanes of a row sit next to each other in one wave, so per-row sums combine with one
// xor-1 exchange and no barrier. Used by the fused descriptor/quadratic-form kernel
// and by the adjoint kernel.
#pragma once

#include "pair.h"

namespace flare {

constexpr int NQ = 8;   // (l, m) indices per lane

// ---- the FP8 form's order of sums ----
// That form's energy pass rounds d~ to about eight bits in two e4m3 parts, so a change in the
// last bit of a component that carries it over a rounding boundary moves it by up to 2^-8 of
// itself: every operation behind d~ is part of the form's results. In the order of the other
// forms its forces moved by 2e-5 to 4e-5 of their norm on gas columns, single ones by 3e-3
// (against 64 bits the form is off by 4.5e-3 in either), where those forms move by 2e-6 at
// most. So this form (template argument FP8) adds the slots in list order, evaluates the
// harmonics as below and contracts them as in b2_half: about 40 instructions more per two
// slots, a step of 200 k atoms 319 -> 320 us, of 1.2 k atoms 98 -> 99 us.
__device__ __forceinline__ void sph_harm_fp8(float x, float y, float z, float* Y) {
#pragma clang fp contract(off)
  const float xx = x * x, yy = y * y, zz = z * z;
  const float dxy = fmaf(-y, y, xx);                 // x^2 - y^2
  const float z4 = fmaf(-y, y, fmaf(4.f, zz, -xx));  // 4 z^2 - x^2 - y^2
  Y[0] = kY0;
  Y[1] = kY1 * y;
  Y[2] = kY1 * z;
  Y[3] = kY1 * x;
  Y[4] = kY2a * x * y;
  Y[5] = kY2a * y * z;
  Y[6] = kY20 * fmaf(-y, y, fmaf(2.f, zz, -xx));
  Y[7] = kY2a * x * z;
  Y[8] = kY22 * dxy;
  Y[9] = kY33 * y * fmaf(3.f, xx, -yy);
  Y[10] = kY32a * x * y * z;
  Y[11] = kY31 * y * z4;
  Y[12] = kY30 * z * fmaf(-3.f, yy, fmaf(2.f, zz, -3.f * xx));
  Y[13] = kY31 * x * z4;
  Y[14] = kY32b * z * dxy;
  Y[15] = kY33 * x * fmaf(-3.f, yy, xx);
}

// c[n][q] += R_n Y_{8h+q} over the neighbours of row R (atom i) inside the cutoff. The lanes
// take the slots in turns (k = 2 m + h): each forms its slot's geometry from the fixed part and
// the displacements (kept in v.geom for the later passes when keep), evaluates the basis once
// and hands the partner R and the partner's half of Y; both then add the two slots, their own
// first (the FP8 form: both the even lane's first).
// All rows of a wave share one slice, so the trip count is uniform across the wave.
// What a slot needs arrives over two dependent loads: the fixed parts are loaded two groups of
// two slots a lane ahead and the neighbours' displacements one, in two register groups that take
// turns (every value is used from the register it was loaded into, so that each wait covers
// only the older group). Loads are unconditional: past the slice they re-read its last slot.
template <bool FP8>
__device__ __forceinline__ void accumulate_half(const SlotView& v, int R, int i, int h, bool keep, float (*c)[NQ]) {
#pragma clang fp contract(off)
  const int S = wave_slice(R);
  const int base = v.slice_base[S];
  const int len = v.slice_base[S + 1] - base;
  if (len <= 0) return;
  const float4 di = v.dlt[i];
  const size_t s0 = (size_t)base * 32 + (R & 31);
  const float4* p = v.d0 + s0;
  float4* to = v.geom + s0;
  auto fixed = [&](int k) { return p[(size_t)min(k + h, len - 1) * 32]; };
  auto moved = [&](const float4& d) { return v.dlt[slot_neighbour(d)]; };
  auto add = [&](int k, float4 g) {
    if (k >= len) return;
    if (k + h >= len) g.w = 0.f;
    else if (keep) to[(size_t)(k + h) * 32] = g;
    const float r = g.w != 0.f ? fabsf(g.w) : v.rc;       // R = 0 at the cutoff, exactly
    float R0[NR], Y[NLM], R1[NR];
    radial(r, v.rc, R0);
    if (FP8) sph_harm_fp8(g.x, g.y, g.z, Y);
    else sph_harm(g.x, g.y, g.z, Y);
#pragma unroll
    for (int n = 0; n < NR; ++n) R1[n] = xor1(R0[n]);
    if (FP8) {
#pragma unroll
      for (int n = 0; n < NR; ++n) {
        const float own = R0[n];
        R0[n] = h ? R1[n] : own;
        R1[n] = h ? own : R1[n];
      }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const float own = h ? Y[NQ + q] : Y[q];
      const float other = xor1(h ? Y[q] : Y[NQ + q]);
      const float y0 = FP8 && h ? other : own, y1 = FP8 && h ? own : other;
#pragma unroll
      for (int n = 0; n < NR; ++n) c[n][q] = fmaf(R1[n], y1, fmaf(R0[n], y0, c[n][q]));
    }
  };
  float4 da[2], ea[2], db[2], eb[2], g[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) da[u] = fixed(2 * u);
#pragma unroll
  for (int u = 0; u < 2; ++u) db[u] = fixed(4 + 2 * u);
#pragma unroll
  for (int u = 0; u < 2; ++u) ea[u] = moved(da[u]);
  for (int k0 = 0;; k0 += 8) {
#pragma unroll
    for (int u = 0; u < 2; ++u) eb[u] = moved(db[u]);
#pragma unroll
    for (int u = 0; u < 2; ++u) g[u] = slot_geom(da[u], ea[u], di, v.rc2);
#pragma unroll
    for (int u = 0; u < 2; ++u) da[u] = fixed(k0 + 8 + 2 * u);
#pragma unroll
    for (int u = 0; u < 2; ++u) add(k0 + 2 * u, g[u]);
    if (k0 + 4 >= len) break;
#pragma unroll
    for (int u = 0; u < 2; ++u) ea[u] = moved(da[u]);
#pragma unroll
    for (int u = 0; u < 2; ++u) g[u] = slot_geom(db[u], eb[u], di, v.rc2);
#pragma unroll
    for (int u = 0; u < 2; ++u) db[u] = fixed(k0 + 12 + 2 * u);
#pragma unroll
    for (int u = 0; u < 2; ++u) add(k0 + 4 + 2 * u, g[u]);
    if (k0 + 8 >= len) break;
  }
}

// One B2 radial pair (a, b) of a single-species block, split between the two lanes of
// the row: lane 0 returns the components l = 0, 1, lane 1 the components l = 2, 3 (the
// lane's half of the packed float4 at 4k). Products c_a,q c_b,q: lane 0 holds l = 0 (q0),
// l = 1 (q1..3) and part of l = 2 (q4..7); lane 1 the rest of l = 2 (q0) and l = 3
// (q1..7). One cross-lane move per pair brings lane 0's part of l = 2 to lane 1.
// FP8: lane 1's l = 2 ends in one fused multiply-add, and with the last channel (last) the two
// first products of each sum come the other way round.
template <bool FP8>
__device__ __forceinline__ float2 b2_half(const float* ca, const float* cb, int h, bool last) {
#pragma clang fp contract(off)
  const bool late = FP8 && last;
  const float p1 = late ? fmaf(ca[1], cb[1], ca[2] * cb[2]) : fmaf(ca[2], cb[2], ca[1] * cb[1]);
  const float p4 = late ? fmaf(ca[4], cb[4], ca[5] * cb[5]) : fmaf(ca[5], cb[5], ca[4] * cb[4]);
  const float v0 = ca[0] * cb[0];
  const float v1 = fmaf(ca[3], cb[3], p1);
  const float v2 = fmaf(ca[7], cb[7], fmaf(ca[6], cb[6], p4));
  const float x = xor1(v2);            // lane 1 receives lane 0's part of l = 2
  return h ? make_float2(FP8 ? fmaf(ca[0], cb[0], x) : v0 + x, v1 + v2) : make_float2(v0, v1);
}

}  // namespace flare
