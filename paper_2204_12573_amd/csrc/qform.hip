// Mapped quadratic forms of the mixed-environment rows (paper, Eq. 1 and Eq. 2 after the
// exact mapping of Section V.B): for the 544-wide descriptor rows D of a bucket,
//   Y = D beta_s (FP32-accurate products in three BF16 parts, see bf16x3.h), e_i = Y_i . D_i,
//   V_i = D_i . Sigma_s D_i, or |L_s^T D_i|^2 with the Cholesky factor of Sigma_s,
//   g_i = (2/|d~_i|) (Y_i - e_i d_i)  (de_i/dd~_i, formed from Y and D by the adjoint kernel).
// The model matrices come split and in fragment order: [K step 17][column block 34][part 3]
// [lane 64] x 8 bf16; the rows are FP32 and split in registers, beside the products (rows
// written split cost 53 MB of writes and half as much again to read for 16 k rows). Columns
// go in pairs of 16-wide blocks: pair m is columns 32 m .. 32 m + 31, and of a lower-
// triangular factor only the K steps >= m of it are non-zero. Two kernels share the work:
//   k_forms544      many rows: a work-group of four waves takes 128 rows x 4 or 5 column
//                   pairs, 32 rows a wave; the matrix fragments of a K step are shared
//                   through LDS (copied there by the loads themselves, two buffers), the
//                   rows' values go to registers one K step ahead
//   k_forms544_few  few rows: a wave takes one 16-row block x one column pair on its own,
//                   three K steps of fragments in flight, no LDS and no barrier; the rows come
//                   already split and in fragment order from the kernel that forms them
//                   (split here they took 14 us in place of 10 for 1 k rows)
// Both form every product, partial sum and row in the same order, so a row's results do
// not depend on which of them ran.
#include <algorithm>

#include "bf16x3.h"
#include "mixed.h"
#include "state.h"

namespace flare {
namespace {

constexpr int NTQ = 256;
constexpr int XNB = ND / 16;                 // 34 column blocks
constexpr int XNP = ND / 32;                 // 17 column pairs
constexpr int XTILES = 4;                    // column tiles of the many-row kernel
constexpr int XTP = 5;                       // pairs of its widest tile

struct XArgs {
  const float* D;        // rows, [rows][544]
  const uint4* D6;       // few rows: the same split, in fragment order
  const int* aor;        // atom of row (-1: padding), or null: rows 0 .. n_given - 1 are given
  int n_given;
  int rows;              // padded rows (a multiple of 128)
  int split_row;         // rows >= split_row belong to the second bucket (Pt centre)
  int mode;              // bit 0: beta part, bit 1: variance part
  int tri;               // the variance part is the Cholesky factor L: V = |d L|^2
  const uint4* W[2];     // per bucket: beta
  const uint4* V[2];     // per bucket: L or Sigma
  float* Y;              // [rows][544] D beta
  float* P;              // [rows][17] V partials of the column pairs
};

// acc += a b over one K step: the six part products, smallest first
__device__ __forceinline__ void mfma6(const bf8 (&a)[3], const bf8 (&b)[3], f4& acc) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[2], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[2], b[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[0], acc, 0, 0, 0);
}

// Rows are filled from the start of their bucket: a 16-row block without an atom in its
// first row holds padding only.
__device__ __forceinline__ bool block_empty(const XArgs& q, int row0) {
  return q.aor ? q.aor[row0] < 0 : row0 >= q.n_given;
}

// Results of one column pair m of one 16-row block (lane (l16, grp): column 16 j + l16 of the
// pair, rows 4 grp + r): Y, or the pair's share of V.
__device__ __forceinline__ void store_pair(const XArgs& q, bool beta, int row0, int m, int lane, const f4 (&acc)[2]) {
  const int l16 = lane & 15, grp = lane >> 4;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = row0 + 4 * grp + r;
    const size_t at = (size_t)row * ND + 32 * m + l16;
    if (beta) {
      q.Y[at] = acc[0][r];
      q.Y[at + 16] = acc[1][r];
    } else {
      float s = q.tri ? fmaf(acc[1][r], acc[1][r], acc[0][r] * acc[0][r])
                      : fmaf(acc[1][r], q.D[at + 16], acc[0][r] * q.D[at]);
      s = sum16(s);
      if (l16 == 0) q.P[(size_t)row * XNP + m] = s;
    }
  }
}

// One wave: 16 rows x one column pair. Fragments of three K steps are in flight (36
// registers each); the waves of a work-group take neighbouring row blocks of one pair, so
// its matrix fragments come from L1. Bound by the latency of the first loads: 17 K steps of
// 12 products are 3.3 k cycles. 256 rows: 6 us, 1 k rows: 10 us; the many-row kernel needs 17
// steps of 1,920 cycles and a barrier whatever the rows (the FP32 one took 62 us).
__global__ __launch_bounds__(NTQ) void k_forms544_few(XArgs q) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nrb = q.rows >> 4;
  const int task = blockIdx.x * 4 + wave;
  const int rb = task % nrb;
  int m = task / nrb;
  const int nbeta = (q.mode & 1) ? XNP : 0;
  if (m >= nbeta + ((q.mode & 2) ? XNP : 0)) return;
  const bool beta = m < nbeta;
  if (!beta) m -= nbeta;
  const int row0 = rb * 16;
  if (block_empty(q, row0)) return;
  const int bk = row0 >= q.split_row ? 1 : 0;
  const uint4* __restrict__ W = (beta ? (bk ? q.W[1] : q.W[0]) : (bk ? q.V[1] : q.V[0])) + (size_t)2 * m * 3 * 64 + lane;
  const uint4* __restrict__ A = q.D6 + (size_t)rb * XKS * 3 * 64 + lane;
  constexpr int PD = 3;
  bf8 a[PD][3], b[PD][2][3];
  auto load = [&](int ks, int u) {
    const int k = min(ks, XKS - 1);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      a[u][t] = __builtin_bit_cast(bf8, A[(k * 3 + t) * 64]);
#pragma unroll
      for (int j = 0; j < 2; ++j) b[u][j][t] = __builtin_bit_cast(bf8, W[(((size_t)k * XNB + j) * 3 + t) * 64]);
    }
  };
  f4 acc[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
  const int ks0 = !beta && q.tri ? m : 0;
#pragma unroll
  for (int u = 0; u < PD; ++u) load(ks0 + u, u);
  for (int ks = ks0; ks < XKS; ks += PD) {
#pragma unroll
    for (int u = 0; u < PD; ++u) {
      if (ks + u < XKS) {
#pragma unroll
        for (int j = 0; j < 2; ++j) mfma6(a[u], b[u][j], acc[j]);
      }
      load(ks + u + PD, u);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  store_pair(q, beta, row0, m, lane, acc);
}

typedef __attribute__((address_space(1))) const void gvoid;
typedef __attribute__((address_space(3))) void lvoid;

// 128 rows x up to five column pairs. Per K step a wave forms 2 x 10 blocks x 6 products
// (1,920 cycles of its SIMD's matrix core) from 4 KB of rows of its own and 30 KB
// of matrix fragments in LDS; two work-groups a CU. Energies and variances of 13,440 rows:
// 70 us, 47 % of the SIMD cycles matrix work (the work-groups' unequal lengths leave 1.5 of 2
// waves on a SIMD on average), against 140 us on FP32 matrix instructions.
__global__ __launch_bounds__(NTQ, 2) void k_forms544(XArgs q) {
  __shared__ __attribute__((aligned(16))) uint4 Bs[2][XTP * 2 * 3 * 64];
  // Work-group g runs on XCD g % 8, which takes every eighth row tile. Its tiles go column
  // tile by column tile, the longest first (a factor's later columns have fewer K steps), so
  // that the second round of work-groups on a CU is the short ones: row tile by row tile
  // left 1.1 of the 2 waves a SIMD can hold on average, 86 us for 13 k rows.
  const int x = blockIdx.x & 7, nrt = q.rows >> 7;
  const int nrx = (nrt - x + 7) >> 3;
  if (nrx <= 0) return;
  const int order = (blockIdx.x >> 3) / nrx;
  const int rt = x + 8 * ((blockIdx.x >> 3) % nrx);
  bool beta = (q.mode & 1) != 0;
  int ct = order;
  if (q.mode == 3) {             // beta 0, variance 0, beta 1, 2, 3, variance 1, 2, 3
    beta = order == 0 || (order >= 2 && order <= 4);
    ct = order < 2 ? 0 : (order <= 4 ? order - 1 : order - 4);
  }
  if (order >= XTILES * (q.mode == 3 ? 2 : 1)) return;
  const int m0 = ct == 0 ? 0 : 4 * ct + 1;          // pairs 0-4, 5-8, 9-12, 13-16
  const int np = ct == 0 ? 5 : 4;
  const int row0 = rt * 128;
  if (block_empty(q, row0)) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int bk = row0 >= q.split_row ? 1 : 0;
  const uint4* __restrict__ W = (beta ? (bk ? q.W[1] : q.W[0]) : (bk ? q.V[1] : q.V[0])) + (size_t)2 * m0 * 3 * 64;
  const bool tri = !beta && q.tri;
  const int ks0 = tri ? m0 : 0;
  const int wrow = row0 + wave * 32;
  const bool idle = block_empty(q, wrow);           // padding rows only: copies, no products
  const float* __restrict__ A = q.D + (size_t)(wrow + (lane & 15)) * ND + 8 * (lane >> 4);
  f4 acc[2][XTP][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int p = 0; p < XTP; ++p)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][p][j] = f4{0.f, 0.f, 0.f, 0.f};
  // the K step's fragments are contiguous in W and in LDS; wave w copies every fourth 1 KB
  auto copy_b = [&](int ks, int buf) {
    const uint4* src = W + (size_t)ks * XNB * 3 * 64 + lane;
    for (int f = wave; f < np * 6; f += 4)
      __builtin_amdgcn_global_load_lds((gvoid*)(src + f * 64), (lvoid*)(&Bs[buf][f * 64]), 16, 0, 0);
  };
  float4 av[2][2];
  bf8 a[2][3];
  auto load_a = [&](int ks) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int t = 0; t < 2; ++t) av[i][t] = *reinterpret_cast<const float4*>(A + (size_t)i * 16 * ND + ks * 32 + 4 * t);
  };
  // all waves' copies of the next K step have landed before any wave reads them (the copies
  // count as vector memory operations, which a barrier alone does not wait for)
  auto copies_done = [] {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  copy_b(ks0, ks0 & 1);
  load_a(ks0);
  copies_done();
  for (int ks = ks0; ks < XKS; ++ks) {
    const int buf = ks & 1;
    const int kn = min(ks + 1, XKS - 1);
    if (ks + 1 < XKS) copy_b(kn, buf ^ 1);
#pragma unroll
    for (int i = 0; i < 2; ++i) split8x3(av[i], a[i][0], a[i][1], a[i][2]);
    load_a(kn);
    if (!idle) {
      // the next pair's fragments are read from LDS while this pair's products run
      bf8 bA[2][3], bB[2][3];
      auto load_b = [&](int p, bf8 (&b)[2][3]) {
        const int pp = min(p, np - 1);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int t = 0; t < 3; ++t) b[j][t] = __builtin_bit_cast(bf8, Bs[buf][((2 * pp + j) * 3 + t) * 64 + lane]);
      };
      load_b(0, bA);
#pragma unroll
      for (int p = 0; p < XTP; ++p) {
        bf8 (&b)[2][3] = (p & 1) ? bB : bA;
        load_b(p + 1, (p & 1) ? bA : bB);
        __builtin_amdgcn_sched_barrier(0);
        if (p >= np || (tri && ks < m0 + p)) continue;
        // the four blocks' products in turn (each accumulator's in the order of mfma6)
#define X_PROD(PA, PB)                                                                                  \
  _Pragma("unroll") for (int i = 0; i < 2; ++i) _Pragma("unroll") for (int j = 0; j < 2; ++j)          \
      acc[i][p][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i][PA], b[j][PB], acc[i][p][j], 0, 0, 0);
        X_PROD(0, 2)
        X_PROD(1, 1)
        X_PROD(0, 1)
        X_PROD(2, 0)
        X_PROD(1, 0)
        X_PROD(0, 0)
#undef X_PROD
      }
    }
    copies_done();
  }
  if (idle) return;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if (i == 1 && block_empty(q, wrow + 16)) break;
#pragma unroll
    for (int p = 0; p < XTP; ++p)
      if (p < np) store_pair(q, beta, wrow + 16 * i, m0 + p, lane, acc[i][p]);
  }
}

void launch_forms544(const XArgs& q, hipStream_t st) {
  const int parts = ((q.mode & 1) ? 1 : 0) + ((q.mode & 2) ? 1 : 0);
  if (q.rows <= FEW_ROWS) {
    const int tasks = (q.rows / 16) * XNP * parts;
    k_forms544_few<<<(tasks + 3) / 4, NTQ, 0, st>>>(q);
  } else {
    const int per_xcd = (q.rows / 128 + 7) / 8;      // row tiles of the fullest XCD
    k_forms544<<<8 * per_xcd * XTILES * parts, NTQ, 0, st>>>(q);
  }
}

// Given vectors in fragment order (rows past n: zeros, as their FP32 copies).
__global__ __launch_bounds__(NTQ) void k_split544(int rows, const float* __restrict__ D, uint4* __restrict__ D6) {
  const int idx = blockIdx.x * NTQ + threadIdx.x;      // (row, packed group of four)
  if (idx >= rows * (ND / 4)) return;
  const int row = idx / (ND / 4), P = idx % (ND / 4);
  store_d6(D6, row, P, reinterpret_cast<const float4*>(D)[idx]);
}

// e_i = Y_i . D_i and V_i from the column pairs' shares (fixed orders), 16 lanes a row, for
// the calls without forces (with them the adjoint kernel forms both on its way to g).
__global__ __launch_bounds__(256) void k_forms544_finish(int rows, int mode, const float* __restrict__ D,
                                                         const float* __restrict__ Y, const float* __restrict__ P,
                                                         const int* __restrict__ aor, int n_given,
                                                         float* __restrict__ e_int, float* __restrict__ v_int,
                                                         float* __restrict__ e_row, float* __restrict__ v_row) {
  const int row = blockIdx.x * 16 + (threadIdx.x >> 4);
  const int L = threadIdx.x & 15;
  if (row >= rows) return;
  const int atom = aor ? aor[row] : (row < n_given ? row : -1);   // no table: given vectors
  if (atom < 0) return;
  if (mode & 2) {
    const float v = mixed_row_variance(P + (size_t)row * XNP, L);
    if (L == 0) {
      v_int[atom] = v;
      v_row[row] = v;
    }
  }
  if (mode & 1) {
    float4 d[NQ4], y[NQ4];
    const float e = mixed_row_energy(reinterpret_cast<const float4*>(D + (size_t)row * ND),
                                     reinterpret_cast<const float4*>(Y + (size_t)row * ND), L, d, y);
    if (L == 0) {
      e_int[atom] = e;
      e_row[row] = e;
    }
  }
}

// Variance of the mixed rows in the split forms, in FP64: V_i = |L_s^T d_i|^2 with the FP64
// Cholesky factor of Sigma_s on v_mfma_f64_16x16x4_f64 (exact products of the FP32 row and
// the FP64 factor, FP64 sums), so the near-cancelling d^T Sigma d keeps FP64 accuracy in the
// form. A wave owns 32 rows (two 16-row blocks, which share every B fragment) and one pair m
// of 16-column blocks of Z = D L: for every K chunk from 2 m on (L[k][n] = 0 for k < n) lane
// (l, q) supplies D[row l][16 kc + 4 q + t] and the fragments L[16 kc + 4 q + t][16 cb + l]
// (fragment order [cb][kc][t][lane]); four independent accumulators per k-step, and the next
// chunk's fragments load while this one runs. Accumulator r of lane (n, q) holds row q + 4 r
// of the block (the FP64 instruction's layout). The pair's sum of squares per row goes to
// P64[row][m]; the pairs are added in a fixed order.
// Bound by the FP64 matrix rate (595 blocks x 8 products of 64 cycles a 32-row block: 62 us
// for 16 k rows). A pair's work falls from 34 chunks to 2, so the pairs go out longest first
// as work units of their own, 95 us (35 us for 4 k rows, 23 us for 128); four-block groups in
// balanced pairs of equal length left three waves on some SIMDs and two on others: 111 us
// (57 us for 4 k rows).
constexpr int XCB = ND / 16;                 // 34 column blocks
typedef double d4 __attribute__((ext_vector_type(4)));

struct VarArgs {
  const float* D;          // [rows][544]
  int rows;                // padded rows (a multiple of 64)
  int split_row;           // rows >= split_row belong to the second bucket (Pt centre)
  const int* aor;          // as XArgs
  int n_given;
  const double* L[2];      // per bucket: fragments of the factor
  double* P64;             // [rows][XNP]
};

constexpr int VRB = 2;                       // 16-row blocks a wave (4: no faster at 16 k rows, 41 : 23 us at 128)
__global__ __launch_bounds__(256) void k_var544_f64(VarArgs q) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nrb = q.rows / (16 * VRB);
  const int task = blockIdx.x * 4 + wave;
  if (task >= nrb * XNP) return;
  const int m = task / nrb;
  const int row0 = (task - m * nrb) * 16 * VRB;
  if (q.aor ? q.aor[row0] < 0 : row0 >= q.n_given) return;     // padding rows only
  const int l16 = lane & 15, grp = lane >> 4;
  // the split between the two buckets falls on a 128-row boundary: one factor per block
  const double* __restrict__ L = (row0 >= q.split_row ? q.L[1] : q.L[0]) + (size_t)2 * m * XCB * 4 * 64 + lane;
  const float* __restrict__ d0 = q.D + (size_t)(row0 + l16) * ND + 4 * grp;
  d4 acc[VRB][2];
#pragma unroll
  for (int i = 0; i < VRB; ++i)
#pragma unroll
    for (int u = 0; u < 2; ++u) acc[i][u] = d4{0.0, 0.0, 0.0, 0.0};
  // chunk 2 m of the pair's second block lies above the diagonal and is stored as zeros
  auto load = [&](int kc, double (&b)[2][4], float4 (&x)[VRB]) {
    const int k = min(kc, XCB - 1);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int t = 0; t < 4; ++t) b[u][t] = L[((size_t)(u * XCB + k) * 4 + t) * 64];
#pragma unroll
    for (int i = 0; i < VRB; ++i) x[i] = *reinterpret_cast<const float4*>(d0 + (size_t)i * 16 * ND + k * 16);
  };
  auto products = [&](const double (&b)[2][4], const float4 (&x)[VRB]) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < VRB; ++i) {
          const float v = t == 0 ? x[i].x : t == 1 ? x[i].y : t == 2 ? x[i].z : x[i].w;
          acc[i][u] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)v, b[u][t], acc[i][u], 0, 0, 0);
        }
  };
  double bA[2][4], bB[2][4];
  float4 xA[VRB], xB[VRB];
  load(2 * m, bA, xA);
  // the chunks of a pair are even in number (34 - 2 m): two per trip, one buffer each
  for (int kc = 2 * m; kc < XCB; kc += 2) {
    load(kc + 1, bB, xB);
    __builtin_amdgcn_sched_barrier(0);
    products(bA, xA);
    load(kc + 2, bA, xA);
    __builtin_amdgcn_sched_barrier(0);
    products(bB, xB);
  }
#pragma unroll
  for (int i = 0; i < VRB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double ss = sum16d(fma(acc[i][1][r], acc[i][1][r], acc[i][0][r] * acc[i][0][r]));
      if (l16 == 0) q.P64[(size_t)(row0 + 16 * i + grp + 4 * r) * XNP + m] = ss;
    }
}

// V of each mixed row from its pair sums, rounded to FP32 once, for the calls without forces.
__global__ __launch_bounds__(256) void k_var544_finish(int rows, const double* __restrict__ P64,
                                                       const int* __restrict__ aor, int n_given,
                                                       float* __restrict__ v_int, float* __restrict__ v_row) {
  const int row = blockIdx.x * 16 + (threadIdx.x >> 4);
  const int L = threadIdx.x & 15;
  if (row >= rows) return;
  const int atom = aor ? aor[row] : (row < n_given ? row : -1);
  if (atom < 0) return;
  const float v = mixed_row_variance(P64 + (size_t)row * XNP, L);
  if (L == 0) {
    v_int[atom] = v;
    v_row[row] = v;
  }
}

void var544_f64(flare_state* s, const float* D, int rows, int split_row, const int* aor, int n_given,
                float* v_int, float* v_row, bool finish) {
  VarArgs q{};
  q.D = D;
  q.rows = rows;
  q.split_row = split_row;
  q.aor = aor;
  q.n_given = n_given;
  q.L[0] = s->model->Lx64[0];
  q.L[1] = s->model->Lx64[1];
  q.P64 = s->Px64;
  k_var544_f64<<<(rows / (16 * VRB) * XNP + 3) / 4, 256, 0, s->stream>>>(q);
  if (finish)
    k_var544_finish<<<(rows + 15) / 16, 256, 0, s->stream>>>(rows, s->Px64, aor, n_given, v_int, v_row);
}

}  // namespace

// Quadratic forms of the mixed-environment rows [r0, r0 + nr) (544-wide, one chunk of the
// workspace: Dx row r - r0). In the split forms the variance runs in FP64 (var544_f64) and
// the products cover beta only. With finish, e and V leave here; otherwise the adjoint kernel
// of the same chunk writes them.
void forms_mixed_chunk(flare_state* s, int r0, int nr, bool want_e, bool want_v, bool finish) {
  if ((!want_e && !want_v) || nr == 0) return;
  StageTimer tm(s, FLARE_T_QFORMX);
  const flare_model* m = s->model;
  const int* aor = s->atom_of_rowx + r0;
  float* e_row = s->e_row + s->rows1 + r0;
  float* v_row = s->v_row + s->rows1 + r0;
  const int split = s->bucket_row0[5] - r0;
  if (want_v && m->var64) {
    var544_f64(s, s->Dx, nr, split, aor, 0, s->v_int, v_row, finish);
    want_v = false;
    if (!want_e) return;
  }
  XArgs q{};
  q.D = s->Dx;
  q.D6 = s->D6x;
  q.aor = aor;
  q.rows = nr;
  q.split_row = split;
  q.mode = (want_e ? 1 : 0) | (want_v ? 2 : 0);
  q.tri = m->vchol ? 1 : 0;
  for (int k = 0; k < 2; ++k) {
    q.W[k] = reinterpret_cast<const uint4*>(m->Wx6[k]);
    q.V[k] = reinterpret_cast<const uint4*>(m->Vx6[k]);
  }
  q.Y = s->Yx;
  q.P = s->Px;
  launch_forms544(q, s->stream);
  if (finish)
    k_forms544_finish<<<(nr + 15) / 16, 256, 0, s->stream>>>(nr, q.mode, s->Dx, s->Yx, s->Px, aor, 0, s->e_int,
                                                             s->v_int, e_row, v_row);
}

// Quadratic forms of given 544-wide vectors (rows 0 .. n-1) with the model of mixed bucket
// `bucket` (4: H centre, 5: Pt centre): e_r = d_r^T beta_s d_r, v_r = d_r^T Sigma_s d_r, by
// the same kernels as the descriptor path. The vectors are copied into the state's padded
// row buffer Dx (zeros past n); scratch: D6x, Yx, Px, Px64, e_row, v_row.
int forms_given_544(flare_state* s, int bucket, int n, const float* d, float* e, float* v) {
  const flare_model* m = s->model;
  for (int c0 = 0; c0 < n; c0 += s->mix_cap) {
    const int nc = std::min(s->mix_cap, n - c0);
    const int rows = (nc + TILE_ROWS - 1) / TILE_ROWS * TILE_ROWS;
    hipError_t err = hipMemcpyAsync(s->Dx, d + (size_t)c0 * ND, (size_t)nc * ND * sizeof(float),
                                    hipMemcpyDeviceToDevice, s->stream);
    if (err == hipSuccess && rows > nc)
      err = hipMemsetAsync(s->Dx + (size_t)nc * ND, 0, (size_t)(rows - nc) * ND * sizeof(float), s->stream);
    if (err != hipSuccess) return (int)err;
    if (rows <= FEW_ROWS)
      k_split544<<<(rows * (ND / 4) + NTQ - 1) / NTQ, NTQ, 0, s->stream>>>(rows, s->Dx, s->D6x);
    // every row of the chunk has the model of `bucket`: the Pt-centre factor from row 0 for
    // bucket 5, the H-centre one throughout for bucket 4
    const int split = bucket == 5 ? 0 : rows;
    XArgs q{};
    q.D = s->Dx;
    q.D6 = s->D6x;
    q.n_given = nc;
    q.rows = rows;
    q.split_row = split;
    q.mode = 3;
    q.tri = m->vchol ? 1 : 0;
    for (int k = 0; k < 2; ++k) {
      q.W[k] = reinterpret_cast<const uint4*>(m->Wx6[k]);
      q.V[k] = reinterpret_cast<const uint4*>(m->Vx6[k]);
    }
    q.Y = s->Yx;
    q.P = s->Px;
    if (m->var64) {
      var544_f64(s, s->Dx, rows, split, nullptr, nc, v + c0, s->v_row, true);
      q.mode = 1;
    }
    launch_forms544(q, s->stream);
    k_forms544_finish<<<(rows + 15) / 16, 256, 0, s->stream>>>(rows, q.mode, s->Dx, s->Yx, s->Px, nullptr, nc, e + c0,
                                                               v + c0, s->e_row, s->v_row);
  }
  return 0;
}

}  // namespace flare
