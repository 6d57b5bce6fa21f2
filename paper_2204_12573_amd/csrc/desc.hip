// Per-atom densities, B2 contraction over m and normalisation (paper, Section V.B).
//
//   c_{(s,n),l,m} = sum_{j in rho_i, s_j = s, r_ij < r_c} R_n(r_ij) Y_lm(r^_ij)
//   d~_{(a,b),l}  = sum_m c_{a,l,m} c_{b,l,m}    (a <= b, packed)
//   d             = d~ / |d~|
//
// This file holds the mixed-environment rows (544 components, 16 lanes per row, see
// mixed.h). Single-species rows are formed inside the fused quadratic-form kernel
// (fused.hip).
// Pair geometry: Delta = [(w_j - w_i) + s*L] + (delta_j - delta_i), the bracket formed in FP64 at
// the list build and kept in FP32, the displacements since then (FP64 differences, kept in FP32)
// added in FP32 (pair.h).
#include "mixed_desc.h"

namespace flare {
namespace {

template <bool EXPORT>
__global__ __launch_bounds__(MTHREADS) void k_desc_mixed(MixedDescArgs q) {
  __shared__ __attribute__((aligned(16))) float lds[MIXED_LDS];
  desc_mixed_block<EXPORT>(q, blockIdx.x, lds);
}

constexpr int NTG = 256;

// Displacement of every atom since the list build, x - xb in FP64, in caller order (the
// loads coalesced), stored in FP32 at the atom's internal index. It must stay within half
// the skin; it is kept in FP32 because it is smaller than half the skin, so its rounding is
// far below that of the pair vectors.
__global__ __launch_bounds__(NTG) void k_disp(int n, const int* __restrict__ inv_perm,
                                              const double* __restrict__ x, const double* __restrict__ y,
                                              const double* __restrict__ z, const double* __restrict__ xb,
                                              float4* __restrict__ dlt, double lim2, int* __restrict__ status) {
  const int a = blockIdx.x * NTG + threadIdx.x;
  if (a >= n) return;
  store_displacement(a, n, x[a], y[a], z[a], xb, inv_perm, dlt, lim2, status);
}

// |d~| of every atom in caller order (0 for an atom without neighbours).
__global__ __launch_bounds__(NTG) void k_export_norms(int n, const int* __restrict__ perm,
                                                      const int* __restrict__ bucket,
                                                      const float* __restrict__ nrm,
                                                      float* __restrict__ norm_out) {
  const int i = blockIdx.x * NTG + threadIdx.x;
  if (i >= n) return;
  norm_out[perm[i]] = bucket[i] < 0 ? 0.f : nrm[i];
}

}  // namespace

void gather_positions(flare_state* s, const double* x, const double* y, const double* z) {
  const int n = s->n_atoms;
  if (n == 0) return;
  const double lim = 0.5 * s->skin;
  k_disp<<<(n + NTG - 1) / NTG, NTG, 0, s->stream>>>(n, s->inv_perm, x, y, z, s->xb, s->dlt, lim * lim,
                                                     s->d_status);
}

MixedDescArgs mixed_desc_args(flare_state* s, int r0, int nr, float* d_out, bool keep) {
  return MixedDescArgs{slot_view(s), s->rows1, r0, s->atom_of_rowx, s->perm, s->Dx, nr <= FEW_ROWS ? s->D6x : nullptr,
                       keep ? s->Cx : nullptr, s->nrm, d_out, keep};
}

void desc_mixed_chunk(flare_state* s, int r0, int nr, bool keep) {
  StageTimer tm(s, FLARE_T_DESCX);
  if (nr > 0)
    k_desc_mixed<false><<<nr / MROWS, MTHREADS, 0, s->stream>>>(mixed_desc_args(s, r0, nr, nullptr, keep));
}

void export_mixed_chunk(flare_state* s, int r0, int nr, float* d_out) {
  StageTimer tm(s, FLARE_T_DESCX);
  if (nr > 0) k_desc_mixed<true><<<nr / MROWS, MTHREADS, 0, s->stream>>>(mixed_desc_args(s, r0, nr, d_out, false));
}

void export_norms(flare_state* s, float* norm_out) {
  const int n = s->n_atoms;
  if (n == 0 || !norm_out) return;
  k_export_norms<<<(n + NTG - 1) / NTG, NTG, 0, s->stream>>>(n, s->perm, s->bucket, s->nrm, norm_out);
}

}  // namespace flare
