// Cell-binned neighbour list and environment classification.
//
// The local environment rho_i is every atom (and periodic image) within the cutoff
// (paper, Section V.B). The list is built with radius r_list = r_cut + skin:
//   1. wrap every position into its cell, w = x - L*floor(x/L), and bin it on a grid
//      of cells >= r_list per axis;
//   2. counting sort by (cell, bin) with a deterministic order inside each bin, which
//      also defines the internal atom order (spatially local);
//   3. per atom, scan the (2K+1)^3 bins around it on the unwrapped bin lattice, so a
//      box with fewer than three bins per axis (or narrower than r_list) visits each
//      (bin, image shift) once; keep (j, s) with |w_j - w_i + s*L|^2 < r_list^2,
//      evaluated in FP64 without fused multiply-add;
//   4. OR the species bits of the neighbours: atoms that see one species only use that
//      species-pair block of the descriptor (the reduction of Section V.B).
// Every buffer has its capacity from flare_state_create. The sizes a build finds (pairs,
// atoms per environment class, rows, slices, slots) are formed on the device in a small
// layout record (d_layout) that the later kernels read; the host waits for the stream once,
// at the end, to read that record and the status words back.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "pair.h"
#include "state.h"

namespace flare {
namespace {

constexpr int NT = 256;

// Layout record of a build (d_layout), formed on the device.
enum {
  LY_PAIRS = 0,      // listed pairs (nl_off[n])
  LY_COUNT = 1,      // [6] atoms per environment bucket
  LY_ROW0 = 7,       // [6] first row of each bucket inside its width class
  LY_ROWS1 = 13,     // padded rows of the 144-wide class
  LY_ROWSX = 14,     // padded rows of the 544-wide class
  LY_SLICES = 15,    // 32-row slices of both classes
  LY_SLOTS32 = 16,   // groups of 32 slots (the slice_base total)
  LY_FLAGS = 17,     // 1: more pairs than the capacity, 2: more slots than the capacity
  LY_STATUS = 18,    // the caller-visible status word raised since it was last read
  LY_N = 19
};
constexpr int BUILD_ASYMMETRIC = 256;   // a pair without its reverse (internal error)
constexpr int BUILD_OVERFLOW = 512;     // more pairs than an int32 prefix holds
constexpr int BUILD_DENSE = 1024;       // some atom has more pairs than PAIR_CACHE

__device__ inline int floor_div(int u, int n) { return u >= 0 ? u / n : -((-u + n - 1) / n); }

// Caller order: wrap into the cell, bin, one 64-byte record per atom, bin counts; the
// positions themselves are kept (xb) as the reference of the per-step displacements.
struct WrapArgs {
  int n;
  const double *x, *y, *z;
  const int32_t* species;
  const int* cell_off;
  int n_cell;
  const CellGrid* grids;
  CallerRec* rec;
  double* xb;
  int* status;
};
__device__ __forceinline__ int wrap_atom(const WrapArgs& q, int a) {
#pragma clang fp contract(off)
  const int n = q.n, n_cell = q.n_cell;
  const int* __restrict__ cell_off = q.cell_off;
  const CellGrid* __restrict__ grids = q.grids;
  const double *__restrict__ x = q.x, *__restrict__ y = q.y, *__restrict__ z = q.z;
  const int32_t* __restrict__ species = q.species;
  CallerRec* __restrict__ rec = q.rec;
  double* __restrict__ xb = q.xb;
  int* __restrict__ status = q.status;
  int lo = 0, hi = n_cell - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (cell_off[mid] <= a) lo = mid;
    else hi = mid - 1;
  }
  const CellGrid g = grids[lo];
  int s = species[a];
  if (s < 0 || s >= NS) atomicOr(status, FLARE_FLAG_SPECIES);
  double p[3] = {x[a], y[a], z[a]};
  double wv[3], ov[3];
  int b[3];
  bool finite = true;
  for (int ax = 0; ax < 3; ++ax) finite = finite && isfinite(p[ax]);
  if (!finite) {
    atomicOr(status, FLARE_FLAG_NONFINITE);
    p[0] = p[1] = p[2] = 0.0;
  }
  for (int ax = 0; ax < 3; ++ax) {
    const double L = g.L[ax];
    const double k = floor(p[ax] / L);
    const double kl = L * k;
    wv[ax] = p[ax] - kl;
    ov[ax] = -kl;
    int bi = (int)floor(wv[ax] * g.inv_h[ax]);
    b[ax] = bi < 0 ? 0 : (bi >= g.nb[ax] ? g.nb[ax] - 1 : bi);
  }
  CallerRec r;
  r.wx = wv[0];
  r.wy = wv[1];
  r.wz = wv[2];
  r.ox = ov[0];
  r.oy = ov[1];
  r.oz = ov[2];
  r.bin = g.bin_base + (b[2] * g.nb[1] + b[1]) * g.nb[0] + b[0];
  r.cell = lo;
  r.pad0 = r.pad1 = 0;
  rec[a] = r;
  xb[a] = p[0];
  xb[(size_t)n + a] = p[1];
  xb[2 * (size_t)n + a] = p[2];
  return r.bin;
}
__global__ __launch_bounds__(NT) void k_wrap_bin(WrapArgs q, int* __restrict__ bin_count) {
  const int a = blockIdx.x * NT + threadIdx.x;
  if (a < q.n) atomicAdd(&bin_count[wrap_atom(q, a)], 1);
}

__global__ __launch_bounds__(NT) void k_bin_scatter(int n, const CallerRec* __restrict__ rec,
                                                    const int* __restrict__ start,
                                                    int* __restrict__ fill,
                                                    int* __restrict__ sorted) {
  const int a = blockIdx.x * NT + threadIdx.x;
  if (a >= n) return;
  const int b = rec[a].bin;
  sorted[start[b] + atomicAdd(&fill[b], 1)] = a;
}

// Internal order: bins in order, inside a bin by caller index (the scatter order is racy: an
// atom's place is the number of smaller indices among its bin's atoms). One caller record (a
// 64-byte line) per atom; the species rides in w.w, so that a neighbour's position and
// species are one load.
struct InternalArgs {
  int n;
  const CallerRec* rec;
  const int32_t* species;
  int *perm, *inv_perm, *sp, *sid, *bin;
  double4* w;
  float4* wf;
  double* off;
};
__device__ __forceinline__ void place_atom(const InternalArgs& q, int a, const CallerRec& r, int i) {
  const int n = q.n;
  q.perm[i] = a;
  q.inv_perm[a] = i;
  const int s = q.species[a];
  const int sc = (s < 0 || s >= NS) ? 0 : s;
  q.sp[i] = sc;
  q.sid[i] = r.cell;
  q.bin[i] = r.bin;
  q.w[i] = make_double4(r.wx, r.wy, r.wz, (double)sc);
  q.wf[i] = make_float4((float)r.wx, (float)r.wy, (float)r.wz, (float)sc);
  q.off[i] = r.ox;
  q.off[(size_t)n + i] = r.oy;
  q.off[2 * (size_t)n + i] = r.oz;
}
__global__ __launch_bounds__(NT) void k_to_internal(InternalArgs q, const int* __restrict__ sorted,
                                                    const int* __restrict__ start) {
  const int t = blockIdx.x * NT + threadIdx.x;
  if (t >= q.n) return;
  const int a = sorted[t];
  const CallerRec r = q.rec[a];
  const int lo = start[r.bin], hi = start[r.bin + 1];
  int i = lo;
  for (int k = lo; k < hi; ++k) i += sorted[k] < a ? 1 : 0;
  place_atom(q, a, r, i);
}

// Row order inside a bucket: by neighbour count, largest first (counts of NCK - 1 and more
// share the last class), ties by internal index. The 32-row slices of the sliced layout
// then hold rows of nearly equal length, so a wave's trip count over its slice (the
// longest row) wastes few lanes. (Measured: ordering only inside 128-row tiles, or inside
// windows of 4096 atoms, keeps more spatial locality for the per-slot gathers but leaves
// enough padding in the slices to cost more in the fused kernel than it saves there.)
// Sort key of an atom in bucket b with count c: b * NCK + (NCK - 1 - min(c, NCK - 1)).
constexpr int NCK = 64;
constexpr int NKEY = NBUCKET * NCK;
__device__ inline int row_key(int b, int c) { return b * NCK + (NCK - 1 - min(c, NCK - 1)); }

// The pair search, 16 lanes an atom. The stencil bins of one (z, y) row and one x image are
// neighbours in the bin order, so their atoms are one contiguous range: a segment. The lanes
// take 16 segments at a time (nine cover a stencil of one bin each way away from the box
// edges), add up their lengths, and then walk the candidates of all of them together, 16 at a
// time; the accepted ones keep the order (z, y, x, bin, place) through a ballot. emit(k, j,
// shift) receives pair k of the atom. The FP32 copies decide every candidate whose FP32
// distance is outside [lo2, hi2) (the band holds the FP32 error, so the decision is the FP64
// one), the FP64 test the rest. Returns the pair count and the species seen.
// (One thread an atom, walking 27 bins through dependent loads, took 58 us for 80 atoms and
// 244 us for 1.0 M.)
constexpr int SL = 16;                       // lanes an atom
constexpr int SA = NT / SL;                  // atoms per work-group

struct PairSearch {
  const CellGrid* grids;
  const int* sid;
  const int* bin;
  const double4* w;
  const float4* wf;
  const int* bstart;
  double rl2;
  float lo2, hi2;
};

template <class Emit>
__device__ __forceinline__ void search_atom(const PairSearch& q, int i, int& cnt_out, int& mask_out, Emit emit) {
#pragma clang fp contract(off)
  const int l = threadIdx.x & (SL - 1);
  const int sub0 = (threadIdx.x & 63) & ~(SL - 1);       // first lane of the group in its wave
  const CellGrid* g = q.grids + q.sid[i];
  const int nbx = g->nb[0], nby = g->nb[1], nbz = g->nb[2];
  const int local = q.bin[i] - g->bin_base;
  const int bx = local % nbx;
  const int by = (local / nbx) % nby;
  const int bz = local / (nbx * nby);
  const int kx = g->K[0], ky = g->K[1], kz = g->K[2], base = g->bin_base;
  const double Lx = g->L[0], Ly = g->L[1], Lz = g->L[2];
  const float lx = (float)Lx, ly = (float)Ly, lz = (float)Lz;
  const float4 wi = q.wf[i];
  const int sx0 = floor_div(bx - kx, nbx);               // images of the x row: sx0 .. sx0 + nsx - 1
  const int nsx = floor_div(bx + kx, nbx) - sx0 + 1;
  const int rows_y = 2 * ky + 1;
  const int nseg = (2 * kz + 1) * rows_y * nsx;
  int cnt = 0, mask = 0;
  for (int e0 = 0; e0 < nseg; e0 += SL) {
    // this lane's segment: first atom, length, image
    const int e = e0 + l;
    int j0 = 0, len = 0, shift = 0;
    if (e < nseg) {
      const int row = e / nsx, sx = sx0 + (e - row * nsx);
      const int rz = row / rows_y;
      const int uz = bz + rz - kz, uy = by + (row - rz * rows_y) - ky;
      const int sz = floor_div(uz, nbz), sy = floor_div(uy, nby);
      const int b0 = base + ((uz - sz * nbz) * nby + (uy - sy * nby)) * nbx;
      j0 = q.bstart[b0 + max(bx - kx - sx * nbx, 0)];
      len = q.bstart[b0 + min(bx + kx - sx * nbx, nbx - 1) + 1] - j0;
      shift = pack_shift(sx, sy, sz);
    }
    int incl = len;
#pragma unroll
    for (int d = 1; d < SL; d <<= 1) {
      const int t = __shfl_up(incl, d, SL);
      if (l >= d) incl += t;
    }
    const int excl = incl - len;
    const int total = __shfl(incl, SL - 1, SL);
    for (int c0 = 0; c0 < total; c0 += SL) {
      const int c = c0 + l;
      // the candidate's segment: the last one that starts at or before it
      int k = 0;
#pragma unroll
      for (int d = SL / 2; d > 0; d >>= 1)
        if (__shfl(excl, k + d, SL) <= c) k += d;
      const int j = __shfl(j0, k, SL) + (c - __shfl(excl, k, SL));
      const int sh = __shfl(shift, k, SL);
      bool in = false;
      int sp = 0;
      if (c < total) {
        int sx, sy, sz;
        unpack_shift(sh, sx, sy, sz);
        const float4 wj = q.wf[j];
        const float fx = (wj.x - wi.x) + (float)sx * lx;
        const float fy = (wj.y - wi.y) + (float)sy * ly;
        const float fz = (wj.z - wi.z) + (float)sz * lz;
        const float r2f = fx * fx + fy * fy + fz * fz;
        in = r2f < q.lo2;
        if (!in && r2f < q.hi2) {
          const double4 wd = q.w[j], wi64 = q.w[i];
          const double dx = (wd.x - wi64.x) + (double)sx * Lx;
          const double dy = (wd.y - wi64.y) + (double)sy * Ly;
          const double dz = (wd.z - wi64.z) + (double)sz * Lz;
          in = dx * dx + dy * dy + dz * dz < q.rl2;
        }
        in = in && !(sh == 0 && j == i);
        sp = wj.w != 0.f ? 1 : 0;
      }
      const unsigned hits = (unsigned)(__ballot(in) >> sub0) & ((1u << SL) - 1u);
      const unsigned pt = (unsigned)(__ballot(in && sp == 1) >> sub0) & ((1u << SL) - 1u);
      if (in) emit(cnt + __popc(hits & ((1u << l) - 1u)), j, sh);
      mask |= (pt ? 2 : 0) | (hits != pt ? 1 : 0);
      cnt += __popc(hits);
    }
  }
  cnt_out = cnt;
  mask_out = mask;
}

// The search keeps the first PAIR_CACHE pairs of atom i at cache[PAIR_CACHE i ...] (j, packed
// shift), so that the pass that writes the list copies them and repeats the search only for
// atoms with more (32 covers every atom of the 1 M-atom H2/Pt(111) cell at r_list 4.7 A, whose
// largest count is 28). Also the atom's environment bucket and the counts of the sort keys in
// its 256-atom block, blk[key * nblk + block].
constexpr int PAIR_CACHE = 32;
// Up to FEW_ATOMS the search and the list run in the forms for few atoms. Search in us, 16
// lanes against one thread an atom: 64 : 72 for a 64 k-atom slab, 97 : 81 for 120 k, 64 : 90
// for 60 k atoms under a gas column, 108 : 95 for 200 k; list with 16 against 64 atoms a
// work-group: 29 : 33 and 51 : 59 for the slabs, 161 : 144 for 800 k atoms under a gas column.
constexpr int FEW_ATOMS = 81920;
constexpr int MANY_AW = 64;

// Up to FEW_ATOMS 16 lanes an atom (blk cleared at the build's start).
__global__ __launch_bounds__(NT) void k_search(int n, PairSearch q, int* __restrict__ cnt_out,
                                               int* __restrict__ bucket, int* __restrict__ blk, int nblk,
                                               int2* __restrict__ cache, int* __restrict__ build_status) {
  const int i = blockIdx.x * SA + threadIdx.x / SL;
  if (i >= n) return;
  int cnt, mask;
  int2* mine = cache + (size_t)i * PAIR_CACHE;
  search_atom(q, i, cnt, mask, [&](int k, int j, int shift) {
    if (k < PAIR_CACHE) mine[k] = make_int2(j, shift);
  });
  if ((threadIdx.x & (SL - 1)) == 0) {
    cnt_out[i] = cnt;
    if (cnt > PAIR_CACHE) atomicOr(build_status, BUILD_DENSE);
    const int b = bucket_of((int)q.w[i].w, mask);
    bucket[i] = b;
    if (b >= 0) atomicAdd(&blk[(size_t)row_key(b, cnt) * nblk + (i >> 8)], 1);
  }
}

// More atoms: one thread an atom, the same segments in the same order, four candidates at a
// time. It spends a tenth of the instructions per candidate (the 16 lanes share few candidates
// in a gas) but waits for one load after the other, so it needs the chip full of atoms.
__global__ __launch_bounds__(NT) void k_search_many(int n, PairSearch q, int* __restrict__ cnt_out,
                                                    int* __restrict__ bucket, int* __restrict__ blk, int nblk,
                                                    int2* __restrict__ cache, int* __restrict__ build_status) {
#pragma clang fp contract(off)
  __shared__ int key_count[NKEY];
  for (int k = threadIdx.x; k < NKEY; k += NT) key_count[k] = 0;
  __syncthreads();
  const int i = blockIdx.x * NT + threadIdx.x;
  if (i < n) {
    const CellGrid g = q.grids[q.sid[i]];
    const int local = q.bin[i] - g.bin_base;
    const int bx = local % g.nb[0];
    const int by = (local / g.nb[0]) % g.nb[1];
    const int bz = local / (g.nb[0] * g.nb[1]);
    const float4 wi = q.wf[i];
    const float lx = (float)g.L[0], ly = (float)g.L[1], lz = (float)g.L[2];
    int2* mine = cache + (size_t)i * PAIR_CACHE;
    int cnt = 0, mask = 0;
    // four positions from j4 on, past the segment's end its last atom again (unused)
    auto load = [&](int j4, int j1, float4 (&wq)[4]) {
      const int last = max(j1 - 1, 0);
#pragma unroll
      for (int u = 0; u < 4; ++u) wq[u] = q.wf[min(j4 + u, last)];
    };
    auto test = [&](const float4 (&wq)[4], int j4, int j1, int sx, int sy, int sz) {
      const float tx = (float)sx * lx, ty = (float)sy * ly, tz = (float)sz * lz;
      const int shift = pack_shift(sx, sy, sz);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = j4 + u;
        const float fx = (wq[u].x - wi.x) + tx;
        const float fy = (wq[u].y - wi.y) + ty;
        const float fz = (wq[u].z - wi.z) + tz;
        const float r2f = fx * fx + fy * fy + fz * fz;
        if (j >= j1 || !(r2f < q.hi2) || (shift == 0 && j == i)) continue;
        if (!(r2f < q.lo2)) {
          const double4 wd = q.w[j], wi64 = q.w[i];
          const double dx = (wd.x - wi64.x) + (double)sx * g.L[0];
          const double dy = (wd.y - wi64.y) + (double)sy * g.L[1];
          const double dz = (wd.z - wi64.z) + (double)sz * g.L[2];
          if (!(dx * dx + dy * dy + dz * dz < q.rl2)) continue;
        }
        if (cnt < PAIR_CACHE) mine[cnt] = make_int2(j, shift);
        mask |= 1 << (int)wq[u].w;
        ++cnt;
      }
    };
    const int sx0 = floor_div(bx - g.K[0], g.nb[0]), sx1 = floor_div(bx + g.K[0], g.nb[0]);
    if (sx0 == sx1 && g.K[1] == 1 && g.K[2] == 1) {
      // nine segments: their ends loaded together
      int j0[9], j1[9], sy[3], sz[3];
#pragma unroll
      for (int rz = 0; rz < 3; ++rz) {
        sz[rz] = floor_div(bz + rz - 1, g.nb[2]);
#pragma unroll
        for (int ry = 0; ry < 3; ++ry) {
          sy[ry] = floor_div(by + ry - 1, g.nb[1]);
          const int b0 = g.bin_base + ((bz + rz - 1 - sz[rz] * g.nb[2]) * g.nb[1] + (by + ry - 1 - sy[ry] * g.nb[1])) * g.nb[0] +
                         bx - sx0 * g.nb[0];
          j0[3 * rz + ry] = q.bstart[b0 - g.K[0]];
          j1[3 * rz + ry] = q.bstart[b0 + g.K[0] + 1];
        }
      }
      // the next four candidates, of this segment or the next one, are on their way while
      // four are tested
      float4 cur[4];
      load(j0[0], j1[0], cur);
#pragma unroll
      for (int r = 0; r < 9; ++r) {
        const int rn = r < 8 ? r + 1 : 8;
        bool more;
        int j4 = j0[r];
        do {
          more = j4 + 4 < j1[r];
          float4 nxt[4];
          load(more ? j4 + 4 : j0[rn], more ? j1[r] : j1[rn], nxt);
          test(cur, j4, j1[r], sx0, sy[r % 3], sz[r / 3]);
#pragma unroll
          for (int u = 0; u < 4; ++u) cur[u] = nxt[u];
          j4 += 4;
        } while (more);
      }
    } else {
      for (int oz = -g.K[2]; oz <= g.K[2]; ++oz) {
        const int sz = floor_div(bz + oz, g.nb[2]);
        for (int oy = -g.K[1]; oy <= g.K[1]; ++oy) {
          const int sy = floor_div(by + oy, g.nb[1]);
          const int b0 = g.bin_base + ((bz + oz - sz * g.nb[2]) * g.nb[1] + (by + oy - sy * g.nb[1])) * g.nb[0];
          for (int sx = sx0; sx <= sx1; ++sx) {
            const int ja = q.bstart[b0 + max(bx - g.K[0] - sx * g.nb[0], 0)];
            const int jb = q.bstart[b0 + min(bx + g.K[0] - sx * g.nb[0], g.nb[0] - 1) + 1];
            for (int j4 = ja; j4 < jb; j4 += 4) {
              float4 wq[4];
              load(j4, jb, wq);
              test(wq, j4, jb, sx, sy, sz);
            }
          }
        }
      }
    }
    cnt_out[i] = cnt;
    if (cnt > PAIR_CACHE) atomicOr(build_status, BUILD_DENSE);
    const int b = bucket_of((int)wi.w, mask);
    bucket[i] = b;
    if (b >= 0) atomicAdd(&key_count[row_key(b, cnt)], 1);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < NKEY; k += NT) blk[(size_t)k * nblk + blockIdx.x] = key_count[k];
}

// Atoms per bucket and the rows of every bucket padded to the 128-row tile (144-wide buckets
// first, then the mixed ones), from the scanned key counts: every work-group that needs them
// adds them up itself (a dozen loads).
struct RowLayout {
  int count[NBUCKET], row0[NBUCKET], rows1, rowsx;
};
__device__ inline RowLayout row_layout(const int* __restrict__ blk_scan, int nblk) {
  RowLayout o;
  int r1 = 0, rx = 0;
#pragma unroll
  for (int b = 0; b < NBUCKET; ++b) {
    const int c = blk_scan[(size_t)(b + 1) * NCK * nblk] - blk_scan[(size_t)b * NCK * nblk];
    const int padded = (c + TILE_ROWS - 1) / TILE_ROWS * TILE_ROWS;
    o.count[b] = c;
    o.row0[b] = b < 4 ? r1 : rx;
    if (b < 4) r1 += padded;
    else rx += padded;
  }
  o.rows1 = r1;
  o.rowsx = rx;
  return o;
}

__device__ __forceinline__ int32_t negated_shift(int32_t v) {
  int sx, sy, sz;
  unpack_shift(v, sx, sy, sz);
  return pack_shift(-sx, -sy, -sz);
}

// Two passes over the atoms that both need only the search and the prefix sums, side by side
// in one launch.
// Work-groups [0, nlist): the list itself, AW atoms a work-group. One thread a pair p =
// (i, j, s), in list order (its atom by bisection in the group's offsets, in LDS), copies it
// from the cache and finds the position of the reverse q = (j, i, -s) inside j's list among
// j's cached pairs, eight a step. The list is symmetric because the FP64 distance test gives
// the same value for both orders (negating a rounded difference is exact). An atom with more
// pairs than the cache is searched again by 16 lanes, and the reverse of a pair that touches
// one is left at -1 for k_rows. Nothing is written when the pairs exceed the capacity.
// AW: 16 atoms, about one pair a thread, when there are few (the kernel is one chain of
// dependent loads); 64 when there are many (fewer groups, offsets shared by more pairs).
// Work-groups from nlist: rows of each bucket in key order (see row_key), 256 atoms a group;
// the rank among equal keys follows the internal index (the scanned key counts of the blocks
// before, then the rank inside the block). The first of them writes the layout record.
template <int AW>
__global__ __launch_bounds__(NT) void k_lists(int n, int nlist, PairSearch q, const int* __restrict__ cnt,
                                              const int* __restrict__ nl_off, const int2* __restrict__ cache,
                                              long long max_pairs, const int* __restrict__ build_status,
                                              int* __restrict__ nl_j, int32_t* __restrict__ nl_s,
                                              int* __restrict__ nl_rev, const int* __restrict__ bucket,
                                              const int* __restrict__ blk_scan, int nblk, int* __restrict__ row_of,
                                              int* __restrict__ aor1, int* __restrict__ aorx,
                                              int* __restrict__ layout) {
  const int pairs = nl_off[n];
  const bool over = (*build_status & BUILD_OVERFLOW) || (long long)pairs > max_pairs;
  if ((int)blockIdx.x < nlist) {
    if (over) return;
    __shared__ int offs[AW + 1];
    const int a0 = blockIdx.x * AW;
    const int na = min(AW, n - a0);
    for (int k = threadIdx.x; k <= na; k += NT) offs[k] = nl_off[a0 + k];
    __syncthreads();
    for (int p = offs[0] + threadIdx.x; p < offs[na]; p += NT) {
      int lo = 0, hi = na;            // largest k with offs[k] <= p
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (offs[mid] <= p) lo = mid;
        else hi = mid;
      }
      if (offs[lo + 1] - offs[lo] > PAIR_CACHE) continue;
      const int2 e = cache[(size_t)(a0 + lo) * PAIR_CACHE + (p - offs[lo])];
      const int len = cnt[e.x];
      const int4* list = reinterpret_cast<const int4*>(cache + (size_t)e.x * PAIR_CACHE);
      const int32_t want = negated_shift(e.y);
      int rev = -1;
      if (len <= PAIR_CACHE)
        for (int k = 0; k < len && rev < 0; k += 8) {
          int4 t[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) t[u] = list[(k >> 1) + u];   // inside the atom's 32 entries
#pragma unroll
          for (int u = 3; u >= 0; --u) {
            if (t[u].z == a0 + lo && t[u].w == want && k + 2 * u + 1 < len) rev = k + 2 * u + 1;
            if (t[u].x == a0 + lo && t[u].y == want && k + 2 * u < len) rev = k + 2 * u;
          }
        }
      nl_j[p] = e.x;
      nl_s[p] = e.y;
      nl_rev[p] = rev;
    }
    if (*build_status & BUILD_DENSE)
      for (int k = threadIdx.x >> 4; k < na; k += SA) {
        const int p0 = offs[k];
        if (offs[k + 1] - p0 <= PAIR_CACHE) continue;
        int c, m;
        search_atom(q, a0 + k, c, m, [&](int pos, int j, int shift) {
          nl_j[p0 + pos] = j;
          nl_s[p0 + pos] = shift;
          nl_rev[p0 + pos] = -1;
        });
      }
    return;
  }
  const int block = blockIdx.x - nlist;
  const RowLayout lay = row_layout(blk_scan, nblk);
  if (block == 0 && threadIdx.x == 0) {
    layout[LY_PAIRS] = pairs;
    for (int b = 0; b < NBUCKET; ++b) {
      layout[LY_COUNT + b] = lay.count[b];
      layout[LY_ROW0 + b] = lay.row0[b];
    }
    layout[LY_ROWS1] = lay.rows1;
    layout[LY_ROWSX] = lay.rowsx;
    layout[LY_SLICES] = (lay.rows1 + lay.rowsx) / 32;
    layout[LY_FLAGS] = over ? 1 : 0;
  }
  __shared__ int keys[NT];
  const int i = block * NT + threadIdx.x;
  const int b = i < n ? bucket[i] : -1;
  const int key = b >= 0 ? row_key(b, cnt[i]) : -1;
  keys[threadIdx.x] = key;
  __syncthreads();
  if (i >= n) return;
  if (b < 0) {
    row_of[i] = -1;
    return;
  }
  int rank = 0;
  for (int k = 0; k < (int)threadIdx.x; ++k) rank += keys[k] == key ? 1 : 0;
  int row0 = 0;
#pragma unroll
  for (int k = 0; k < NBUCKET; ++k) row0 = b == k ? lay.row0[k] : row0;
  const int row = row0 + (blk_scan[(size_t)key * nblk + block] - blk_scan[(size_t)b * NCK * nblk]) + rank;
  row_of[i] = row;
  if (b < 4) aor1[row] = i;
  else aorx[row] = i;
}

// Row R of atom i: 144-wide rows R = row_of[i], mixed rows R = rows1 + row_of[i].
__device__ inline int global_row(int b, int r, int rows1) { return b < 4 ? r : rows1 + r; }

// Work-groups [0, nrows): per-row copies of the atom's pair count and cell (padding rows: 0,
// 0) and the length of each 32-row slice, the largest pair count of its rows (zero for the
// slices past the build's, so that the prefix over them ends at the build's total).
// Work-groups from nrows, only when some atom has more pairs than the cache: the reverse
// positions left open by k_lists, from the complete list; a pair (i, j) with i <= j is searched
// for in j's list and both positions are kept (a pair of an atom with its own image by both its
// lanes, with the same two values). 1.8 ms for 200 k atoms with 110 pairs each, where every pair
// searched for, an entry a step, took 4.0.
__global__ __launch_bounds__(NT) void k_rows(int row_max, int nrows, const int* __restrict__ layout,
                                             const int* __restrict__ build_status, const int* __restrict__ aor1,
                                             const int* __restrict__ aorx, const int* __restrict__ cnt,
                                             const int* __restrict__ sid, int* __restrict__ cnt_row,
                                             int* __restrict__ sid_row, int* __restrict__ slice_len, int n,
                                             const int* __restrict__ nl_off, const int* __restrict__ nl_j,
                                             const int32_t* __restrict__ nl_s, int* __restrict__ nl_rev) {
  if ((int)blockIdx.x < nrows) {
    const int R = blockIdx.x * NT + threadIdx.x;
    const int rows1 = layout[LY_ROWS1], rows = rows1 + layout[LY_ROWSX];
    int c = 0;
    if (R < rows) {
      const int i = R < rows1 ? aor1[R] : aorx[R - rows1];
      c = i >= 0 ? cnt[i] : 0;
      cnt_row[R] = c;
      sid_row[R] = i >= 0 ? sid[i] : 0;
    }
#pragma unroll
    for (int d = 16; d > 0; d >>= 1) c = max(c, __shfl_xor(c, d, 32));
    if ((threadIdx.x & 31) == 0 && R < row_max) slice_len[R >> 5] = c;
    return;
  }
  if (!(*build_status & BUILD_DENSE) || layout[LY_FLAGS]) return;
  const int i = (blockIdx.x - nrows) * SA + (threadIdx.x >> 4);
  if (i >= n) return;
  const int p0 = nl_off[i], own = nl_off[i + 1] - p0;
  for (int k = threadIdx.x & 15; k < own; k += 16) {
    const int j = nl_j[p0 + k];
    if (j < i) continue;            // found by the partner's lane
    if (own <= PAIR_CACHE && cnt[j] <= PAIR_CACHE) continue;
    const int32_t want = negated_shift(nl_s[p0 + k]);
    const int q0 = nl_off[j], q1 = nl_off[j + 1];
    int found = -1;
    // four entries a step, their loads together
    for (int m = q0; m < q1 && found < 0; m += 4) {
      int jj[4];
      int32_t ss[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int at = min(m + u, q1 - 1);
        jj[u] = nl_j[at];
        ss[u] = nl_s[at];
      }
#pragma unroll
      for (int u = 3; u >= 0; --u)
        if (jj[u] == i && ss[u] == want) found = min(m + u, q1 - 1);
    }
    if (found >= 0) {
      nl_rev[p0 + k] = found - q0;
      nl_rev[found] = k;
    }
  }
}

// Row of every atom in caller order and the slot of its first pair in internal order (-1:
// no listed pair, no row); the first work-item also records the slots of the build.
struct AtomRowArgs {
  int n;
  const int *bucket, *row_of;
  int* layout;
  const int* perm;
  int slice_max;
  long long slot_cap;
  int *row_caller, *slot0;
};
__device__ __forceinline__ void slots_total(const AtomRowArgs& q, int groups) {
  q.layout[LY_SLOTS32] = groups;
  if ((long long)groups * 32 > q.slot_cap) q.layout[LY_FLAGS] |= 2;
}
__device__ __forceinline__ void atom_row(const AtomRowArgs& q, int i, const int* slice_base) {
  const int b = q.bucket[i];
  const int R = b < 0 ? -1 : global_row(b, q.row_of[i], q.layout[LY_ROWS1]);
  q.row_caller[q.perm[i]] = R;
  q.slot0[i] = R < 0 ? -1 : slot_of(slice_base, R, 0);
}
__global__ __launch_bounds__(NT) void k_atom_rows(AtomRowArgs q, const int* __restrict__ slice_base) {
  const int i = blockIdx.x * NT + threadIdx.x;
  if (i == 0) slots_total(q, slice_base[q.slice_max]);
  if (i < q.n) atom_row(q, i, slice_base);
}

// The sliced pair layout in one pass, a work-group per 32-row slice: thread (h, l) of 8 x 32
// takes the slots (slice_base[S] + k) * 32 + l for k = h, h + 8, ... of row R = 32 S + l, so
// every store is coalesced and the gathers of eight positions of a row are in flight at
// once. A slot of a listed pair p = (i, j, s) gets the fixed part of the pair vector
// (w_j - w_i) + s*L (FP64, stored FP32) with j and its species in .w, and the slot of
// its reverse pair: slot0[j] + 32 rev[p], rev[p] being the reverse pair's position in j's
// list. Per pair this gathers two things of the neighbour, w[j] and slot0[j]. Every other
// slot of the slice is padding: pointing at itself, with no neighbour (for every step of
// the list's life).
__global__ __launch_bounds__(NT) void k_slots(const int* __restrict__ layout, const int* __restrict__ aor1,
                                              const int* __restrict__ aorx, const int* __restrict__ nl_off,
                                              const int* __restrict__ nl_j, const int32_t* __restrict__ nl_s,
                                              const int* __restrict__ nl_rev, const int* __restrict__ slot0,
                                              const int* __restrict__ slice_base, const double4* __restrict__ w,
                                              const int* __restrict__ sid, const CellGrid* __restrict__ grids,
                                              int* __restrict__ slot_rev, float4* __restrict__ slot_d0,
                                              int* __restrict__ status) {
#pragma clang fp contract(off)
  if (layout[LY_FLAGS]) return;
  const int S = blockIdx.x;
  if (S >= layout[LY_SLICES]) return;
  const int rows1 = layout[LY_ROWS1];
  const int l = threadIdx.x & 31, h = threadIdx.x >> 5;
  const int R = S * 32 + l;
  const int i = R < rows1 ? aor1[R] : aorx[R - rows1];
  const int base = slice_base[S], len = slice_base[S + 1] - base;
  int p0 = 0, own = 0;
  double4 wi = make_double4(0.0, 0.0, 0.0, 0.0);
  double L[3] = {0.0, 0.0, 0.0};
  if (i >= 0) {
    p0 = nl_off[i];
    own = nl_off[i + 1] - p0;
    wi = w[i];
    const CellGrid* g = grids + sid[i];
    L[0] = g->L[0];
    L[1] = g->L[1];
    L[2] = g->L[2];
  }
  for (int k = h; k < len; k += NT / 32) {
    const int slot = (base + k) * 32 + l;
    if (k < own) {
      const int p = p0 + k;
      const int j = nl_j[p];
      const int q = nl_rev[p];
      int sx, sy, sz;
      unpack_shift(nl_s[p], sx, sy, sz);
      const int sj = slot0[j];
      const double4 wj = w[j];
      int rs = slot;
      if (q < 0) atomicOr(status, BUILD_ASYMMETRIC);
      else rs = sj + 32 * q;
      const double dx = (wj.x - wi.x) + (double)sx * L[0];
      const double dy = (wj.y - wi.y) + (double)sy * L[1];
      const double dz = (wj.z - wi.z) + (double)sz * L[2];
      slot_rev[slot] = rs;
      slot_d0[slot] = make_float4((float)dx, (float)dy, (float)dz, __int_as_float(slot_code(j, wj.w != 0.0 ? 1 : 0)));
    } else {
      slot_rev[slot] = slot;            // padding slots point at themselves
      slot_d0[slot] = pad_slot();
    }
  }
}

// The fills of a build in one launch: up to ten (array, count, value) segments, every
// work-item striding over each of them.
struct ClearSeg {
  int* p;
  long long n;
  int v;
};
struct ClearArgs {
  ClearSeg seg[10];
  int nseg;
  int* status;    // [0] the caller-visible word, [1] the build's; the layout record follows
  int* layout;
};
__device__ __forceinline__ void clear_all(const ClearArgs& a, long long t, long long stride) {
  if (t == 0) {
    // the caller-visible status word moves to the layout record (read by the host at the end
    // of the build) and is cleared: no flag of the ended interval is lost
    for (int k = 0; k < LY_N; ++k) a.layout[k] = 0;
    a.layout[LY_STATUS] = a.status[0];
    a.status[0] = 0;
    a.status[1] = 0;
  }
  for (int k = 0; k < a.nseg; ++k) {
    int* __restrict__ p = a.seg[k].p;
    const long long n = a.seg[k].n;
    const int v = a.seg[k].v;
    for (long long i = t; i < n; i += stride) p[i] = v;
  }
}
__global__ __launch_bounds__(NT) void k_clear(ClearArgs a) {
  clear_all(a, (long long)blockIdx.x * NT + threadIdx.x, (long long)gridDim.x * NT);
}

// Builds of up to ONE_ATOMS atoms and ONE_BINS bins (what LDS holds beside the order): the passes that need little more than a
// launch each run as phases of one work-group, with bin counts and the bin order in LDS. k_first:
// the fills, wrap and bin, scan, scatter, internal order (five launches); k_last_rows: the slice
// scan and the atoms' rows (two). Each launch taken out is 3 us of the stream and as much of the
// host's time; one CU pays for it with about 10 us a thousand atoms. A whole build in us, general
// passes -> here: 72 atoms 85 -> 60, 540 85 -> 66, 1,215 86 -> 73, 1,980 86 -> 80, but 3,024
// 86 -> 90, 4,032 88 -> 102.
constexpr int NT1 = 1024;
constexpr int ONE_ATOMS = 2048, ONE_BINS = 8192, ONE_PER = ONE_ATOMS / NT1;

// Exclusive prefix of one value a thread over the work-group; total: the sum over all.
__device__ __forceinline__ int group_scan(int v, int* wsum, int& total) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int incl = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int t = __shfl_up(incl, d, 64);
    if (lane >= d) incl += t;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  int before = 0;
  total = 0;
  for (int k = 0; k < NT1 / 64; ++k) {
    if (k < w) before += wsum[k];
    total += wsum[k];
  }
  return before + incl - v;
}

__global__ __launch_bounds__(NT1) void k_first(ClearArgs c, WrapArgs q, InternalArgs o, int nbins,
                                               int* __restrict__ bin_start) {
  __shared__ int start[ONE_BINS];       // counts, then first places, then (scattered) ends
  __shared__ int sorted[ONE_ATOMS];
  __shared__ int wsum[NT1 / 64];
  const int t = threadIdx.x;
  clear_all(c, t, NT1);
  for (int b = t; b < nbins; b += NT1) start[b] = 0;
  __syncthreads();
  int bin[ONE_PER];
#pragma unroll
  for (int u = 0; u < ONE_PER; ++u) {
    const int a = u * NT1 + t;
    bin[u] = a < q.n ? wrap_atom(q, a) : -1;
    if (bin[u] >= 0) atomicAdd(&start[bin[u]], 1);
  }
  __syncthreads();
  const int per = (nbins + NT1 - 1) / NT1, base = t * per;
  int sum = 0, total;
  for (int k = base; k < min(base + per, nbins); ++k) sum += start[k];
  int run = group_scan(sum, wsum, total);
  for (int k = base; k < min(base + per, nbins); ++k) {
    const int m = start[k];
    start[k] = run;
    bin_start[k] = run;
    run += m;
  }
  if (t == 0) bin_start[nbins] = total;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < ONE_PER; ++u)
    if (bin[u] >= 0) sorted[atomicAdd(&start[bin[u]], 1)] = u * NT1 + t;
  __syncthreads();
  // inside a bin by caller index (the scatter order is racy), as in k_to_internal
#pragma unroll
  for (int u = 0; u < ONE_PER; ++u) {
    if (bin[u] < 0) continue;
    const int a = u * NT1 + t;
    const int lo = bin[u] > 0 ? start[bin[u] - 1] : 0, hi = start[bin[u]];
    int i = lo;
    for (int k = lo; k < hi; ++k) i += sorted[k] < a ? 1 : 0;
    place_atom(o, a, q.rec[a], i);
  }
}

__global__ __launch_bounds__(NT1) void k_last_rows(AtomRowArgs q, const int* __restrict__ slice_len,
                                                   int* __restrict__ slice_base) {
  __shared__ int base[NT1];
  __shared__ int wsum[NT1 / 64];
  const int t = threadIdx.x;
  int total;
  const int first = group_scan(t < q.slice_max ? slice_len[t] : 0, wsum, total);
  base[t] = first;
  if (t < q.slice_max) slice_base[t] = first;
  if (t == 0) {
    slice_base[q.slice_max] = total;
    slots_total(q, total);
  }
  __syncthreads();
  for (int i = t; i < q.n; i += NT1) atom_row(q, i, base);
}
static_assert((ONE_ATOMS + NBUCKET * TILE_ROWS + 31) / 32 <= NT1, "a slice a thread");

inline int grid_of(long long n) { return (int)((n + NT - 1) / NT); }

#define HIPCHK(call)                                                     \
  do {                                                                   \
    hipError_t e_ = (call);                                              \
    if (e_ != hipSuccess) {                                              \
      set_error(std::string(#call) + ": " + hipGetErrorString(e_));      \
      return e_ == hipErrorOutOfMemory ? FLARE_E_OOM : FLARE_E_HIP;      \
    }                                                                    \
  } while (0)

}  // namespace

int list_key_count() { return NKEY; }
int list_pair_cache() { return PAIR_CACHE; }
int list_layout_words() { return LY_N; }

int build_list(flare_state* s, const double* x, const double* y, const double* z,
               const int32_t* species) {
  const int n = s->n_atoms;
  hipStream_t st = s->stream;
  const int nc = s->n_struct;
  const int nbins = s->n_bins;
  const int nblk = grid_of(n);
  // reduction tasks: contiguous internal ranges of one cell, at most 2048 atoms each (one
  // work-group per task); cell c owns tasks [first_task[c], first_task[c + 1])
  s->tasks.clear();
  s->longest_task = 0;
  s->first_task.assign(nc + 1, 0);
  for (int c = 0; c < nc; ++c) {
    s->first_task[c] = (int)s->tasks.size();
    const int a = s->struct_off[c], b = s->struct_off[c + 1];
    s->longest_task = std::max(s->longest_task, std::min(b - a, 2048));
    if (a == b) s->tasks.push_back({c, a, a});
    for (int k = a; k < b; k += 2048) s->tasks.push_back({c, k, std::min(b, k + 2048)});
  }
  s->first_task[nc] = (int)s->tasks.size();
  if ((int)s->tasks.size() > s->task_cap) {
    set_error("more reduction tasks than the state holds");
    return FLARE_E_CAPACITY;
  }
  // the per-cell host data through the pinned stage in one copy: grids, offsets, tasks, task
  // ranges (the device copies stand in the same order, see flare_state_create)
  char* hs = s->h_stage;
  const size_t b_grid = nc * sizeof(CellGrid), b_off = (nc + 1) * sizeof(int);
  const size_t b_task = s->tasks.size() * sizeof(RedTask), b_first = (nc + 1) * sizeof(int);
  std::memcpy(hs, s->grids.data(), b_grid);
  std::memcpy(hs + b_grid, s->struct_off.data(), b_off);
  std::memcpy(hs + b_grid + b_off, s->tasks.data(), b_task);
  std::memcpy(hs + b_grid + b_off + b_task, s->first_task.data(), b_first);
  s->d_grids = reinterpret_cast<CellGrid*>(s->d_stage);
  s->d_struct_off = reinterpret_cast<int*>(s->d_stage + b_grid);
  s->d_tasks = reinterpret_cast<RedTask*>(s->d_stage + b_grid + b_off);
  s->d_first_task = reinterpret_cast<int*>(s->d_stage + b_grid + b_off + b_task);
  HIPCHK(hipMemcpyAsync(s->d_stage, hs, b_grid + b_off + b_task + b_first, hipMemcpyHostToDevice, st));
  // the build checks its inputs in a word of its own (d_status[1]); the caller-visible
  // word d_status[0] keeps what the per-step calls raised until k_clear moves it
  int* bst = s->d_status + 1;
  s->d_layout = s->d_status + 16;
  // rows of this many atoms: every bucket's padding included
  const int row_max = std::min(s->row_cap, (n + NBUCKET * TILE_ROWS + 31) / 32 * 32);
  const int slice_max = row_max / 32;
  const bool one = n > 0 && n <= ONE_ATOMS && nbins <= ONE_BINS;
  const WrapArgs wq{n, x, y, z, species, s->d_struct_off, nc, s->d_grids, s->crec, s->xb, bst};
  const InternalArgs io{n, s->crec, species, s->perm, s->inv_perm, s->sp, s->sid, s->bin, s->w, s->wf, s->off};
  {
    // everything the build starts from: its status word and layout record, the bin and key
    // counters, no atom in any row, zero energies, variances and norms (atoms without a
    // listed pair keep them)
    ClearArgs c{};
    c.status = s->d_status;
    c.layout = s->d_layout;
    auto seg = [&](int* p, long long cnt, int v) { c.seg[c.nseg++] = ClearSeg{p, cnt, v}; };
    if (!one) {
      seg(s->bin_count, (long long)nbins + 1, 0);
      seg(s->bin_fill, (long long)nbins + 1, 0);
    }
    if (n <= FEW_ATOMS) seg(s->blk_bucket, (long long)NKEY * nblk, 0);
    seg(s->atom_of_row1, row_max, -1);
    seg(s->atom_of_rowx, row_max, -1);
    seg(reinterpret_cast<int*>(s->e_int), n, 0);
    seg(reinterpret_cast<int*>(s->v_int), n, 0);
    seg(reinterpret_cast<int*>(s->nrm), n, 0);
    long long longest = 1;
    for (int k = 0; k < c.nseg; ++k) longest = std::max(longest, c.seg[k].n);
    if (one) k_first<<<1, NT1, 0, st>>>(c, wq, io, nbins, s->bin_start);
    else k_clear<<<(int)std::min<long long>(grid_of(longest), 2048), NT, 0, st>>>(c);
  }
  if (!one) {
    if (n > 0) k_wrap_bin<<<grid_of(n), NT, 0, st>>>(wq, s->bin_count);
    scan_exclusive(s->bin_count, s->bin_start, nbins, s->scan_scratch, st);
    if (n > 0) {
      k_bin_scatter<<<grid_of(n), NT, 0, st>>>(n, s->crec, s->bin_start, s->bin_fill, s->sorted);
      k_to_internal<<<grid_of(n), NT, 0, st>>>(io, s->sorted, s->bin_start);
    }
  }
  const double rl2 = s->r_list * s->r_list;
  // Band of the FP32 first test. Wrapped coordinates lie in [0, W] (W the largest box side),
  // image shifts are at most K box sides (K the largest stencil half-width), formed in FP32
  // from the rounded side (within 2 u K W), u = 2^-24. A candidate near the list radius has
  // every FP32 pair-vector component within e = u ((3 + 3 K) W + 2 r_list) of the FP64 one, so the FP32 |Delta|^2 is within
  // e (2 sqrt(3) r_list + 3 e) + 4 u r_list^2 of the FP64 value; the band is twice that.
  double wmax = 0.0;
  int kmax = 1;
  for (const CellGrid& g : s->grids)
    for (int ax = 0; ax < 3; ++ax) {
      wmax = std::max(wmax, g.L[ax]);
      kmax = std::max(kmax, g.K[ax]);
    }
  const double u32 = std::ldexp(1.0, -24);
  const double e32 = u32 * ((3.0 + 3.0 * kmax) * wmax + 2.0 * s->r_list);
  const double band = 2.0 * (e32 * (2.0 * std::sqrt(3.0) * s->r_list + 3.0 * e32) + 4.0 * u32 * rl2);
  const float lo2 = std::nextafter((float)(rl2 - band), -INFINITY);
  const float hi2 = std::nextafter((float)(rl2 + band), INFINITY);
  const PairSearch q{s->d_grids, s->sid, s->bin, s->w, s->wf, s->bin_start, rl2, lo2, hi2};
  const bool many = n > FEW_ATOMS;
  const int ngroup = (n + SA - 1) / SA;          // work-groups of 16 atoms
  if (many)
    k_search_many<<<nblk, NT, 0, st>>>(n, q, s->nl_cnt, s->bucket, s->blk_bucket, nblk, s->pair_cache, bst);
  else if (n > 0)
    k_search<<<ngroup, NT, 0, st>>>(n, q, s->nl_cnt, s->bucket, s->blk_bucket, nblk, s->pair_cache, bst);
  scan_exclusive2(s->nl_cnt, s->nl_off, n, s->blk_bucket, s->blk_bucket_scan, NKEY * nblk, s->scan_scratch, bst,
                  BUILD_OVERFLOW, st);
  const int nlist = many ? (n + MANY_AW - 1) / MANY_AW : ngroup;
  auto lists = many ? k_lists<MANY_AW> : k_lists<SA>;
  lists<<<nlist + std::max(nblk, 1), NT, 0, st>>>(n, nlist, q, s->nl_cnt, s->nl_off, s->pair_cache, s->max_pairs, bst,
                                                  s->nl_j, s->nl_s, s->nl_rev, s->bucket, s->blk_bucket_scan, nblk,
                                                  s->row_of, s->atom_of_row1, s->atom_of_rowx, s->d_layout);
  const int nrows = grid_of(row_max);
  k_rows<<<nrows + ngroup, NT, 0, st>>>(row_max, nrows, s->d_layout, bst, s->atom_of_row1, s->atom_of_rowx, s->nl_cnt,
                                       s->sid, s->cnt_row, s->sid_row, s->slice_len, n, s->nl_off, s->nl_j, s->nl_s,
                                       s->nl_rev);
  const AtomRowArgs ar{n, s->bucket, s->row_of, s->d_layout, s->perm, slice_max, s->slot_cap, s->row_caller, s->slot0};
  if (one) {
    k_last_rows<<<1, NT1, 0, st>>>(ar, s->slice_len, s->slice_base);
  } else {
    scan_exclusive(s->slice_len, s->slice_base, slice_max, s->scan_scratch, st);
    k_atom_rows<<<std::max(nblk, 1), NT, 0, st>>>(ar, s->slice_base);
  }
  k_slots<<<slice_max, NT, 0, st>>>(s->d_layout, s->atom_of_row1, s->atom_of_rowx, s->nl_off, s->nl_j, s->nl_s,
                                    s->nl_rev, s->slot0, s->slice_base, s->w, s->sid, s->d_grids, s->slot_rev,
                                    s->slot_d0, bst);
  HIPCHK(hipMemcpyAsync(s->h_info, s->d_status, (16 + LY_N) * sizeof(int), hipMemcpyDeviceToHost, st));
  HIPCHK(hipGetLastError());
  HIPCHK(hipStreamSynchronize(st));      // the build's one wait
  const int* L = s->h_info + 16;
  s->flags_at_build = L[LY_STATUS];
  s->flags_pending |= L[LY_STATUS];
  const int flags = s->h_info[1];
  if (flags & FLARE_FLAG_SPECIES) {
    set_error("species index outside [0, n_species)");
    return FLARE_E_SPECIES;
  }
  if (flags & FLARE_FLAG_NONFINITE) {
    set_error("non-finite position");
    return FLARE_E_NONFINITE;
  }
  if (L[LY_FLAGS] & 1) {
    set_error((flags & BUILD_OVERFLOW) || L[LY_PAIRS] < 0
                  ? std::string("list needs more than 2^31 pairs")
                  : "list needs " + std::to_string(L[LY_PAIRS]) + " pairs, state holds " +
                        std::to_string(s->max_pairs));
    return FLARE_E_CAPACITY;
  }
  if (L[LY_FLAGS] & 2) {
    set_error("sliced pair layout needs " + std::to_string(32LL * L[LY_SLOTS32]) + " slots, state holds " +
              std::to_string(s->slot_cap));
    return FLARE_E_CAPACITY;
  }
  if (flags & BUILD_ASYMMETRIC) {
    set_error("internal: neighbour list is not symmetric");
    return FLARE_E_HIP;
  }
  s->n_pairs = L[LY_PAIRS];
  for (int b = 0; b < NBUCKET; ++b) {
    s->bucket_count[b] = L[LY_COUNT + b];
    s->bucket_row0[b] = L[LY_ROW0 + b];
  }
  s->rows1 = L[LY_ROWS1];
  s->rowsx = L[LY_ROWSX];
  return FLARE_OK;
}

}  // namespace flare
