// Pair data shared by the descriptor and adjoint kernels: the per-step geometry of a slot of
// the sliced layout. It is formed where the densities are, and kept per slot for the adjoint
// terms and the virial. (A kernel of its own for it read the fixed part and wrote the geometry
// for the densities to read again: 85 us of 990 a step of 1.0 M atoms, where the fused kernel
// now takes 43 us longer; 3 us of launch for few atoms.)
#pragma once

#include "basis.h"
#include "state.h"

namespace flare {

struct PairGeom {
  float r, ux, uy, uz;
};

// The slice of row R, read as a wave-uniform (scalar) value: every caller's wave covers
// rows of one 32-row slice, so all its active lanes have the same R / 32.
__device__ __forceinline__ int wave_slice(int R) { return __builtin_amdgcn_readfirstlane(R >> 5); }

// The .w word of a slot's fixed part d0: the neighbour's internal index and species, negative
// for padding (whose index reads as 0, an atom that exists).
__host__ __device__ inline int slot_code(int j, int species) { return (j << 1) | species; }
constexpr int PAD_SLOT = (int)0x80000000u;
__device__ __forceinline__ float4 pad_slot() { return make_float4(0.f, 0.f, 0.f, __int_as_float(PAD_SLOT)); }
__device__ __forceinline__ int slot_neighbour(const float4& d0) {
  return (int)(((unsigned)__float_as_int(d0.w) << 1) >> 2);
}

// Geometry of one listed pair at the current positions. The pair vector is split as
//   Delta = [(w_j - w_i) + s*L] + (delta_j - delta_i),
// the bracket fixed at the list build (d0: FP64, stored rounded to FP32) and the displacements
// since the build added in FP32. Kept when |Delta|^2 < r_c^2, returned as (u^, r) with the sign
// of r carrying the neighbour species; zero outside the cutoff, at
// zero distance and for padding.
__device__ __forceinline__ float4 slot_geom(const float4& d0, const float4& dj, const float4& di, float rc2) {
#pragma clang fp contract(off)
  const int code = __float_as_int(d0.w);
  const float fx = d0.x + (dj.x - di.x), fy = d0.y + (dj.y - di.y), fz = d0.z + (dj.z - di.z);
  const float r2 = fmaf(fz, fz, fmaf(fy, fy, fx * fx));
  if (code < 0 || !(r2 > 0.f && r2 < rc2)) return make_float4(0.f, 0.f, 0.f, 0.f);
  const float r = sqrtf(r2);
  const float inv = 1.f / r;
  return make_float4(fx * inv, fy * inv, fz * inv, code & 1 ? r : -r);
}

__device__ __forceinline__ bool unpack_geom(const float4& g, PairGeom& pg, int& sp) {
  pg.ux = g.x;
  pg.uy = g.y;
  pg.uz = g.z;
  pg.r = fabsf(g.w);
  sp = g.w > 0.f ? 1 : 0;
  return g.w != 0.f;
}

}  // namespace flare
