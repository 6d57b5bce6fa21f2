// FP32 values as three BF16 parts: x = x0 + x1 + x2 holds all 24 significant bits exactly
// (x0 and x1 round the remainder of the previous parts to 8 bits, the remainders are exact
// in FP32, and the last one has at most 8 bits, so its BF16 pattern is the upper half of
// its FP32 pattern). Of the nine part products of two such values the six with a part-index
// sum <= 2 are formed on v_mfma_f32_16x16x32_bf16 (exact products, FP32 accumulation); the
// dropped x1 w2 + x2 w1 + x2 w2 are below 2^-23 |x||w|, the size of one FP32 rounding.
#pragma once

#include "common.h"

namespace flare {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef unsigned int u4v __attribute__((ext_vector_type(4)));

// two FP32 values to a packed BF16 pair (round to nearest even), and back
__device__ __forceinline__ unsigned int pk_bf16(float a, float b) {
  return __builtin_bit_cast(unsigned int, __builtin_convertvector((f2v){a, b}, bf2));
}
__device__ __forceinline__ float bf16_lo(unsigned int p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float bf16_hi(unsigned int p) { return __builtin_bit_cast(float, p & 0xffff0000u); }

// the three parts of two FP32 values, each a packed BF16 pair
__device__ __forceinline__ void split2x3(float a, float b, unsigned int& p0, unsigned int& p1, unsigned int& p2) {
  p0 = pk_bf16(a, b);
  const float ra = a - bf16_lo(p0), rb = b - bf16_hi(p0);
  p1 = pk_bf16(ra, rb);
  const float sa = ra - bf16_lo(p1), sb = rb - bf16_hi(p1);
  p2 = __builtin_amdgcn_perm(__builtin_bit_cast(unsigned int, sb), __builtin_bit_cast(unsigned int, sa), 0x07060302u);
}

__device__ __forceinline__ void split8x3(const float4 (&u)[2], bf8& x0, bf8& x1, bf8& x2) {
  const float v[8] = {u[0].x, u[0].y, u[0].z, u[0].w, u[1].x, u[1].y, u[1].z, u[1].w};
  u4v p0, p1, p2;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    unsigned int q0, q1, q2;
    split2x3(v[2 * t], v[2 * t + 1], q0, q1, q2);
    p0[t] = q0;
    p1[t] = q1;
    p2[t] = q2;
  }
  x0 = __builtin_bit_cast(bf8, p0);
  x1 = __builtin_bit_cast(bf8, p1);
  x2 = __builtin_bit_cast(bf8, p2);
}

// ---- few 544-wide rows in fragment order ----
// D6: [16-row block][K step 17][part 3][lane 64] x 8 bf16, lane l holding row l % 16 and
// k = 32 step + 8 (l / 16) .. + 7: the A operand of one MFMA is one contiguous 1 KB load.
constexpr int XKS = ND / 32;                 // 17 K steps

// components 4 P .. 4 P + 3 of row `row`, split, to their places in D6
__device__ __forceinline__ void store_d6(uint4* __restrict__ D6, int row, int P, const float4& o) {
  const int k = 4 * P;
  const int lane = (row & 15) + 16 * ((k & 31) >> 3);
  uint2* p = reinterpret_cast<uint2*>(D6 + ((size_t)((row >> 4) * XKS + (k >> 5)) * 3 * 64 + lane)) + ((k >> 2) & 1);
  uint2 v[3];
  split2x3(o.x, o.y, v[0].x, v[1].x, v[2].x);
  split2x3(o.z, o.w, v[0].y, v[1].y, v[2].y);
#pragma unroll
  for (int t = 0; t < 3; ++t) p[t * 128] = v[t];
}

}  // namespace flare
