// Mixed-environment rows (both species among the neighbours, 544 components) with 16
// lanes per row: a work-group of 256 threads owns 16 rows, all of one 32-row slice. Lane L =
// s*8 + n of a row accumulates the density channel c_{(s,n), lm} for all 16 (l, m) over the
// row's slots (paper, Section V.B); the channels then meet in LDS, where the B2 contraction
// reads them, and go to the chunk's workspace for the adjoint transform u = G^ c and the pair
// terms. Densities of all 16 channels of a row sit at cidx(a, lm) of the row's block; the Pt
// channels are shifted by 8 floats so that H and Pt reads of one row fall in different banks.
#pragma once

#include "basis.h"
#include "pair.h"

namespace flare {

constexpr int MROWS = 16;                  // rows per work-group
constexpr int MTHREADS = MROWS * 16;       // threads per work-group
constexpr int MSTRIDE = 16 * NLM + 16;     // floats per row, in LDS (4 rows of a wave: distinct banks) and in Cx

__device__ __forceinline__ int cidx(int a, int lm) { return a * NLM + (a >> 3) * 8 + lm; }

// Densities c[lm] of channel L of every row of the work-group, c = sum over the row's slots of
// R_{L & 7}(r) Y_lm(r^) for neighbours of species L >> 3. Slots go in groups of 16: each lane
// forms the geometry of one of them (kept in v.geom for the later
// passes when keep) and evaluates its basis into LDS (16 radial values, the other species' eight
// zero, and 16 harmonics), then every lane adds the 16 slots in order to its channel. (Each
// lane evaluating the whole basis of every slot for its one channel did 1.7 k vector
// instructions a row group where this does 0.6 k: 42.5 -> 37.6 us for 16 k rows of slabs, with the
// rows written once in FP32 where they are many.)
constexpr int PBS = 32;                    // LDS floats per slot
__device__ __forceinline__ void mixed_densities(const SlotView& v, int R, int i, int rl, int L, bool keep,
                                                float* __restrict__ bs, float (&c)[NLM]) {
  const int S = wave_slice(R);
  const int base = v.slice_base[S];
  const int len = v.slice_base[S + 1] - base;
  const size_t s0 = (size_t)base * 32 + (R & 31);
  auto fixed = [&](int k) { return k < len ? v.d0[s0 + (size_t)k * 32] : pad_slot(); };
  const float4 di = i >= 0 ? v.dlt[i] : make_float4(0.f, 0.f, 0.f, 0.f);
  float4 d0 = fixed(L), d1 = fixed(16 + L);
  float4 dj = v.dlt[slot_neighbour(d0)];
  float* mine = bs + (rl * 16 + L) * PBS;
  const float* row = bs + rl * 16 * PBS;
#pragma unroll
  for (int lm = 0; lm < NLM; ++lm) c[lm] = 0.f;
  for (int k0 = 0; k0 < len; k0 += 16) {
    const float4 g = slot_geom(d0, dj, di, v.rc2);
    if (keep && k0 + L < len) v.geom[s0 + (size_t)(k0 + L) * 32] = g;
    d0 = d1;
    dj = v.dlt[slot_neighbour(d0)];
    d1 = fixed(k0 + 32 + L);
    PairGeom pg;
    int sp;
    float Rn[NR], Y[NLM];
    if (unpack_geom(g, pg, sp)) {
      radial(pg.r, v.rc, Rn);
      sph_harm(pg.ux, pg.uy, pg.uz, Y);
    } else {
#pragma unroll
      for (int n = 0; n < NR; ++n) Rn[n] = 0.f;
#pragma unroll
      for (int lm = 0; lm < NLM; ++lm) Y[lm] = 0.f;
    }
    float4* m4 = reinterpret_cast<float4*>(mine);
    const float h = sp ? 0.f : 1.f, t = sp ? 1.f : 0.f;     // exact: the other species' values are zeros
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      m4[u] = make_float4(h * Rn[4 * u], h * Rn[4 * u + 1], h * Rn[4 * u + 2], h * Rn[4 * u + 3]);
      m4[2 + u] = make_float4(t * Rn[4 * u], t * Rn[4 * u + 1], t * Rn[4 * u + 2], t * Rn[4 * u + 3]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) m4[4 + u] = make_float4(Y[4 * u], Y[4 * u + 1], Y[4 * u + 2], Y[4 * u + 3]);
    __syncthreads();
    const int m = min(16, len - k0);
#pragma unroll 2
    for (int k = 0; k < m; ++k) {
      const float rn = row[k * PBS + L];
      const float4* y4 = reinterpret_cast<const float4*>(row + k * PBS + 16);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float4 y = y4[u];
        c[4 * u] = fmaf(rn, y.x, c[4 * u]);
        c[4 * u + 1] = fmaf(rn, y.y, c[4 * u + 1]);
        c[4 * u + 2] = fmaf(rn, y.z, c[4 * u + 2]);
        c[4 * u + 3] = fmaf(rn, y.w, c[4 * u + 3]);
      }
    }
    __syncthreads();
  }
}

// The 16 lanes of a mixed row hold its 136 groups of four components as group L + 16 q of
// lane L. Energy of the row from its descriptor d and y = beta d, in a fixed order (all 16
// lanes get the sum).
constexpr int NQ4 = (ND / 4 + 15) / 16;    // 9
__device__ __forceinline__ float mixed_row_energy(const float4* __restrict__ d4, const float4* __restrict__ y4, int L,
                                                  float4 (&d)[NQ4], float4 (&y)[NQ4]) {
#pragma unroll
  for (int k = 0; k < NQ4; ++k) {
    const int P4 = L + 16 * k;
    d[k] = P4 < ND / 4 ? d4[P4] : make_float4(0.f, 0.f, 0.f, 0.f);
    y[k] = P4 < ND / 4 ? y4[P4] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float e = 0.f;
#pragma unroll
  for (int k = 0; k < NQ4; ++k)
    e = fmaf(d[k].w, y[k].w, fmaf(d[k].z, y[k].z, fmaf(d[k].y, y[k].y, fmaf(d[k].x, y[k].x, e))));
  return sum16(e);
}
// Variance of the row from the shares of its 17 column pairs (FP64 ones summed in FP64 and
// rounded once).
__device__ __forceinline__ float mixed_row_variance(const float* __restrict__ p, int L) {
  return sum16(p[L] + (L == 0 ? p[16] : 0.f));
}
__device__ __forceinline__ float mixed_row_variance(const double* __restrict__ p, int L) {
  return (float)sum16d(p[L] + (L == 0 ? p[16] : 0.0));
}

// Packed B2 pair of channels a and b (either order) of a 544-wide row: (H,H) pairs 0..35
// (na <= nb, row-major), (H,Pt) pairs 36..99 (row-major, H channel first), (Pt,Pt) pairs
// 100..135.
__device__ __forceinline__ int mixed_pair_index(int a, int b) {
  const int lo = a < b ? a : b, hi = a < b ? b : a;
  const int nl = lo & 7, nh = hi & 7;
  if ((lo >> 3) != (hi >> 3)) return NP1 + nl * NR + nh;
  return (lo >> 3 ? NP1 + NX : 0) + nl * NR - nl * (nl - 1) / 2 + (nh - nl);
}

}  // namespace flare
