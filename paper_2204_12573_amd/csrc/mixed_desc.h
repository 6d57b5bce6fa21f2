// Descriptors of the mixed-environment rows (paper, Section V.B): one work-group's 16 rows.
// Launched as a kernel of its own (desc.hip), or beside the single-species rows when there
// are few (fused.hip).
#pragma once

#include "bf16x3.h"
#include "mixed.h"
#include "state.h"

namespace flare {

struct MixedDescArgs {
  SlotView v;
  int rows1, r0;
  const int* atom_of_row;    // of the mixed class
  const int* perm;
  float* D;                  // the chunk's workspace, row - r0
  uint4* D6;                 // the same split, in fragment order, or null
  float* Cx;                 // densities, or null (an evaluation without energies has no adjoint)
  float* nrm_out;
  float* d_out;              // caller order, or null
  bool keep_geom;            // with Cx
};

// LDS of a work-group: the slots' basis values, then the channels, then (export) finished rows
constexpr int MIXED_LDS = MROWS * 16 * PBS;
static_assert(MROWS * MSTRIDE <= MIXED_LDS && MROWS / 2 * ND <= MIXED_LDS, "one block of LDS for all three");

// One mixed row per 16 lanes (mixed.h): channel densities into LDS, then the 136 B2 channel
// pairs spread over the row's lanes, the norm summed in FP64 across the lanes, and the
// normalised row written as float4 per pair: into the chunk's workspace D (row - r0, the
// densities beside it in Cx; few rows also split, in D6), or (EXPORT) into d_out at the atom's
// caller index, the workspace left alone.
template <bool EXPORT>
__device__ __forceinline__ void desc_mixed_block(const MixedDescArgs& q, int block, float* __restrict__ lds) {
#pragma clang fp contract(off)
  const int rl = threadIdx.x >> 4, L = threadIdx.x & 15;
  const int local = block * MROWS + rl;
  const int row = q.r0 + local;
  const int i = q.atom_of_row[row];
  float c[NLM];
  mixed_densities(q.v, q.rows1 + row, i, rl, L, q.keep_geom, lds, c);     // padding rows: empty slots, zeros
  float* crow = lds + rl * MSTRIDE;
#pragma unroll
  for (int lm = 0; lm < NLM; ++lm) crow[cidx(L, lm)] = c[lm];
  __syncthreads();
  if (!EXPORT && q.Cx) {
    float4* to = reinterpret_cast<float4*>(q.Cx + (size_t)block * MROWS * MSTRIDE);
    for (int k = threadIdx.x; k < MROWS * MSTRIDE / 4; k += MTHREADS) to[k] = reinterpret_cast<const float4*>(lds)[k];
  }
  // lane L takes the channel pairs {L, (L + k) mod 16}, k = 0 .. 7, and of k = 8 the lanes
  // below 8 (each unordered pair once): its own channel stays in registers
  constexpr int NQP = 9;
  float4 d[NQP];
  double nrm2 = 0.0;
#pragma unroll
  for (int k = 0; k < NQP; ++k) {
    d[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (k < 8 || L < 8) {
      const float4* y4 = reinterpret_cast<const float4*>(crow + cidx((L + k) & 15, 0));
      float y[NLM];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float4 t = y4[u];
        y[4 * u] = t.x; y[4 * u + 1] = t.y; y[4 * u + 2] = t.z; y[4 * u + 3] = t.w;
      }
      const float d0 = c[0] * y[0];
      float d1 = c[1] * y[1], d2 = c[4] * y[4], d3 = c[9] * y[9];
#pragma unroll
      for (int lm = 2; lm < 4; ++lm) d1 = fmaf(c[lm], y[lm], d1);
#pragma unroll
      for (int lm = 5; lm < 9; ++lm) d2 = fmaf(c[lm], y[lm], d2);
#pragma unroll
      for (int lm = 10; lm < 16; ++lm) d3 = fmaf(c[lm], y[lm], d3);
      d[k] = make_float4(d0, d1, d2, d3);
      nrm2 += (double)fmaf(d0, d0, d1 * d1) + (double)fmaf(d2, d2, d3 * d3);
    }
  }
  nrm2 = sum16d(nrm2);                    // the row's 16 lanes form one DPP row
  if (nrm2 < 0x1p-60) {
    // a row whose only neighbours inside the cutoff are just inside it has components down to
    // 1e-27, which FP32 holds, but not their squares: squared in FP64 (all 16 lanes together)
    nrm2 = 0.0;
#pragma unroll
    for (int k = 0; k < NQP; ++k) {
      const double d0 = d[k].x, d1 = d[k].y, d2 = d[k].z, d3 = d[k].w;
      nrm2 += fma(d0, d0, d1 * d1) + fma(d2, d2, d3 * d3);
    }
    nrm2 = sum16d(nrm2);
  }
  const float nrm = (float)sqrt(nrm2);
  const float scale = nrm > 0.f ? 1.f / nrm : 0.f;
  if (!EXPORT) {
    float4* out = reinterpret_cast<float4*>(q.D + (size_t)local * ND);
#pragma unroll
    for (int k = 0; k < NQP; ++k) {
      if (k < 8 || L < 8) {
        const int P = mixed_pair_index(L, (L + k) & 15);
        const float4 o = make_float4(d[k].x * scale, d[k].y * scale, d[k].z * scale, d[k].w * scale);
        out[P] = o;
        if (q.D6) store_d6(q.D6, local, P, o);
      }
    }
  } else if (q.d_out) {
    // The lanes' pairs are scattered over the row, so it leaves through LDS in whole lines, eight
    // rows at a time (each pair stored from its lane, to the workspace too: the descriptors of
    // 1,500 cells of 64 atoms in 262 us in place of 208, of 256 cells of 80 in 75 in place of
    // 62; the workspace's rows stay in L2 and do not gain by it)
    float4* rows = reinterpret_cast<float4*>(lds);
    for (int half = 0; half < 2; ++half) {
      __syncthreads();                    // the channels, or the first eight rows, have been read
      if ((rl >> 3) == half) {
#pragma unroll
        for (int k = 0; k < NQP; ++k)
          if (k < 8 || L < 8)
            rows[(rl & 7) * (ND / 4) + mixed_pair_index(L, (L + k) & 15)] =
                make_float4(d[k].x * scale, d[k].y * scale, d[k].z * scale, d[k].w * scale);
      }
      __syncthreads();
      for (int k = threadIdx.x; k < MROWS / 2 * (ND / 4); k += MTHREADS) {
        const int r = k / (ND / 4), a = q.atom_of_row[q.r0 + block * MROWS + half * (MROWS / 2) + r];
        if (a >= 0) reinterpret_cast<float4*>(q.d_out)[(size_t)q.perm[a] * (ND / 4) + (k - r * (ND / 4))] = rows[k];
      }
    }
  }
  if (L == 0 && i >= 0) q.nrm_out[i] = nrm;
}

// the arguments for rows [r0, r0 + nr) of the mixed class (desc.hip); keep: geometry and
// densities are left for the adjoint (unasked the densities are 18 MB of stores for 16 k rows:
// the norms of 1,500 cells of 64 atoms 173 us in place of 157)
MixedDescArgs mixed_desc_args(flare_state* s, int r0, int nr, float* d_out, bool keep);

}  // namespace flare
