// Outputs in the caller's atom order, per-cell reductions and the velocity-Verlet halves.
//
// Per-cell energy E = sum_i e_i is accumulated in FP64 with Neumaier compensation, over
// fixed atom ranges in a fixed order (deterministic for given e_i). The per-cell
// maximum uncertainty is the largest sigma_i = sqrt(max(V_i, 0)).
#include "state.h"

namespace flare {
namespace {

constexpr int NT = 256;

__device__ inline void two_sum_add(double& s, double& c, double x) {
  const double t = s + x;
  if (fabs(s) >= fabs(x)) c += (s - t) + x;
  else c += (x - t) + s;
  s = t;
}

// Everything after the forms, in two launches whose work-groups do one of two jobs each (the
// four passes as launches of their own took 4 x 3-5 us of every small step):
//   k_outputs_rows   rows: F_i = sum_k w(i,k) - sum_k w_in(slot(i,k)), the first sum (the
//                    row's own pair terms) formed by the adjoint as f_own, the second over
//                    the row's own pairs k < count in slot order (deterministic), written with
//                    e_i as one 16-byte record per row
//                    tasks: compensated FP64 sum of e and max of sigma over a reduction task
//   k_outputs_atoms  atoms (caller order): each reads its row's record and variance and writes
//                    every requested output (zeros without a row), with the second half of a
//                    velocity-Verlet step when asked for
//                    cells: the tasks of a cell folded in a fixed tree; with a monitor the
//                    running maximum of sigma and the count above the threshold
struct OutArgs {
  int row_groups, task_groups, atom_groups, cells;   // work-groups (cells: one wave each)
  int rows, n, want_f;
  const int* slice_base;
  const float4* f_own;
  const float4* w_in;
  const int* cnt_row;
  const int* sid_row;
  const double* cell_scale;
  const float* e_row;
  float4* row_out;
  // tasks and cells
  const RedTask* tasks;
  const int* bucket;
  const float* e_int;
  const float* v_int;
  int want_e, want_s;
  double* red_e;
  float* red_s;
  const int* first_task;
  double* e_struct;
  float* sigma_max;
  float thr;
  float* run_max;
  int* over;
  int* status;
  // atoms
  const int* row_caller;
  const float* v_row;
  float* e_atom;
  float *fx, *fy, *fz;
  float* var_atom;
  float* sigma_atom;
  // the second half (null: outputs only)
  double *vx, *vy, *vz;
  const int32_t* species;
  double h0, h1;
};

__device__ __forceinline__ void reduce_task(const OutArgs& a, int task) {
  __shared__ double ss[NT], sc[NT];
  __shared__ float sm[NT];
  const RedTask tk = a.tasks[task];
  double s = 0.0, c = 0.0;
  float mx = 0.f;
  for (int i = tk.begin + threadIdx.x; i < tk.end; i += NT) {
    if (a.bucket[i] < 0) continue;
    if (a.want_e) two_sum_add(s, c, (double)a.e_int[i]);
    if (a.want_s) mx = fmaxf(mx, sqrtf(fmaxf(a.v_int[i], 0.f)));
  }
  ss[threadIdx.x] = s;
  sc[threadIdx.x] = c;
  sm[threadIdx.x] = mx;
  __syncthreads();
  for (int h = NT / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) {
      double s2 = ss[threadIdx.x], c2 = sc[threadIdx.x] + sc[threadIdx.x + h];
      two_sum_add(s2, c2, ss[threadIdx.x + h]);
      ss[threadIdx.x] = s2;
      sc[threadIdx.x] = c2;
      sm[threadIdx.x] = fmaxf(sm[threadIdx.x], sm[threadIdx.x + h]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    a.red_e[2 * task] = ss[0];
    a.red_e[2 * task + 1] = sc[0];
    a.red_s[task] = sm[0];
  }
}

__global__ __launch_bounds__(NT) void k_outputs_rows(OutArgs a) {
  if ((int)blockIdx.x >= a.row_groups) {
    reduce_task(a, blockIdx.x - a.row_groups);
    return;
  }
  const int R = xcd_remap(blockIdx.x, a.row_groups) * NT + threadIdx.x;
  if (R >= a.rows) return;
  float sx = 0.f, sy = 0.f, sz = 0.f;
  if (a.want_f) {
    const int base = a.slice_base[R >> 5], len = a.cnt_row[R];   // the row's own pairs (no padding)
    const float4* wp = a.w_in + (size_t)base * 32 + (R & 31);
    float rx = 0.f, ry = 0.f, rz = 0.f;
    int k = 0;
    // four loads in flight at a time; the sums stay in slot order
    for (; k + 4 <= len; k += 4) {
      float4 wr[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) wr[u] = wp[(size_t)(k + u) * 32];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        rx += wr[u].x;
        ry += wr[u].y;
        rz += wr[u].z;
      }
    }
    for (; k < len; ++k) {
      const float4 wr = wp[(size_t)k * 32];
      rx += wr.x;
      ry += wr.y;
      rz += wr.z;
    }
    const float4 fo = a.f_own[R];
    sx = fo.x - rx;
    sy = fo.y - ry;
    sz = fo.z - rz;
    if (a.cell_scale) {
      const float k = (float)a.cell_scale[a.sid_row[R]];
      sx *= k;
      sy *= k;
      sz *= k;
    }
  }
  a.row_out[R] = make_float4(sx, sy, sz, a.e_row[R]);
}

// One wave per cell: its tasks [first_task[c], first_task[c + 1]) are folded by the 64 lanes in
// a fixed stride, then combined in a fixed tree (deterministic).
constexpr int NC = 64;

__device__ __forceinline__ void reduce_cell(const OutArgs& a, int cell) {
  const int t = threadIdx.x & (NC - 1);
  double s = 0.0, c = 0.0;
  float mx = 0.f;
  for (int k = a.first_task[cell] + t; k < a.first_task[cell + 1]; k += NC) {
    two_sum_add(s, c, a.red_e[2 * k]);
    c += a.red_e[2 * k + 1];
    mx = fmaxf(mx, a.red_s[k]);
  }
#pragma unroll
  for (int h = NC / 2; h > 0; h >>= 1) {
    const double so = __shfl_down(s, h, NC), co = __shfl_down(c, h, NC);
    const float mo = __shfl_down(mx, h, NC);
    c += co;
    two_sum_add(s, c, so);
    mx = fmaxf(mx, mo);
  }
  if (t == 0) {
    if (a.e_struct) a.e_struct[cell] = s + c;
    if (a.sigma_max) a.sigma_max[cell] = mx;
    if (a.run_max) {
      a.run_max[cell] = fmaxf(a.run_max[cell], mx);
      if (mx > a.thr) {
        a.over[cell] += 1;
        atomicOr(a.status, FLARE_FLAG_UNCERTAIN);
      }
    }
  }
}

__global__ __launch_bounds__(NT) void k_outputs_atoms(OutArgs o) {
  if ((int)blockIdx.x >= o.atom_groups) {
    const int cell = (blockIdx.x - o.atom_groups) * (NT / NC) + threadIdx.x / NC;
    if (cell < o.cells) reduce_cell(o, cell);
    return;
  }
  const int a = blockIdx.x * NT + threadIdx.x;
  if (a >= o.n) return;
  // all loads ahead of the stores
  const int R = o.row_caller[a];
  double ux = 0.0, uy = 0.0, uz = 0.0, h = 0.0;
  if (o.vx) {
    h = o.species[a] == 0 ? o.h0 : o.h1;
    ux = o.vx[a];
    uy = o.vy[a];
    uz = o.vz[a];
  }
  float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
  float v = 0.f;
  if (R >= 0) {
    r = o.row_out[R];
    if (o.var_atom || o.sigma_atom) v = o.v_row[R];
  }
  if (o.e_atom) o.e_atom[a] = r.w;
  if (o.fx) {
    o.fx[a] = r.x;
    o.fy[a] = r.y;
    o.fz[a] = r.z;
  }
  if (o.var_atom) o.var_atom[a] = v;
  if (o.sigma_atom) o.sigma_atom[a] = sqrtf(fmaxf(v, 0.f));
  if (o.vx) {
    o.vx[a] = ux + h * (double)r.x;
    o.vy[a] = uy + h * (double)r.y;
    o.vz[a] = uz + h * (double)r.z;
  }
}

// Virial of one reduction task (a contiguous internal atom range of one cell): per atom
// the nine products over its own pairs in slot order, summed in FP32; then the atoms of
// the task in FP64 in a fixed order. The cell's W = -sum_p Delta_p (x) w_p runs over all its
// pairs; the reverse q of p has Delta_q = -Delta_p and w_in(slot p) = w_q, so relabelling the
// sum gives W = sum_p Delta_p (x) w_in(slot p), which each atom forms from its own slots
// (Delta = r u from the geometry). red_w [tasks][9] holds the task sums.
// An order of its own for every task, whatever the work-group's size: the atoms go in groups of
// 64, group g taking atoms 64 g + 1024 k, one a lane; each 16 lanes are summed in a fixed tree,
// and these sums in order.
constexpr int VG = 16;                       // groups of a task
template <int NV>
__global__ __launch_bounds__(NV) void k_virial_tasks(const RedTask* __restrict__ tasks,
                                                     const int* __restrict__ bucket,
                                                     const int* __restrict__ row_of, int rows1,
                                                     const int* __restrict__ slice_base,
                                                     const float4* __restrict__ geom,
                                                     const float4* __restrict__ w_in,
                                                     const int* __restrict__ cnt,
                                                     double* __restrict__ red_w) {
  __shared__ double sw[VG * 4][9];
  const RedTask tk = tasks[blockIdx.x];
  const int groups = min(VG, (tk.end - tk.begin + 63) / 64);
  for (int g = threadIdx.x >> 6; g < groups; g += NV / 64) {
    double acc[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) acc[c] = 0.0;
    for (int i = tk.begin + g * 64 + (threadIdx.x & 63); i < tk.end; i += VG * 64) {
      const int b = bucket[i];
      if (b < 0) continue;
      const int R = b < 4 ? row_of[i] : rows1 + row_of[i];
      const int base = slice_base[R >> 5], len = cnt[i];
      float va[9];
#pragma unroll
      for (int c = 0; c < 9; ++c) va[c] = 0.f;
      const size_t s0 = (size_t)base * 32 + (R & 31);
      for (int k0 = 0; k0 < len; k0 += 4) {
        // four slots' loads together (past the list its last slot again, unused)
        float4 gq[4], wq[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const size_t slot = s0 + (size_t)min(k0 + u, len - 1) * 32;
          gq[u] = geom[slot];
          wq[u] = w_in[slot];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (k0 + u >= len) break;
          const float r = fabsf(gq[u].w);      // 0 outside the cutoff: no contribution
          const float d[3] = {r * gq[u].x, r * gq[u].y, r * gq[u].z};
          const float ww[3] = {wq[u].x, wq[u].y, wq[u].z};
#pragma unroll
          for (int x = 0; x < 3; ++x)
#pragma unroll
            for (int y = 0; y < 3; ++y) va[3 * x + y] += d[x] * ww[y];
        }
      }
#pragma unroll
      for (int c = 0; c < 9; ++c) acc[c] += (double)va[c];
    }
#pragma unroll
    for (int c = 0; c < 9; ++c) acc[c] = sum16d(acc[c]);
    if ((threadIdx.x & 15) == 0)
#pragma unroll
      for (int c = 0; c < 9; ++c) sw[g * 4 + ((threadIdx.x >> 4) & 3)][c] = acc[c];
  }
  __syncthreads();
  if (threadIdx.x < 9) {
    double t = 0.0;
    for (int k = 0; k < 4 * groups; ++k) t += sw[k][threadIdx.x];
    red_w[(size_t)blockIdx.x * 9 + threadIdx.x] = t;
  }
}

__global__ __launch_bounds__(NC) void k_virial_cells(const double* __restrict__ red_w,
                                                     const int* __restrict__ first_task,
                                                     double* __restrict__ out) {
  __shared__ double sw[9][NC];
  const int cell = blockIdx.x, t = threadIdx.x;
  double acc[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) acc[c] = 0.0;
  for (int k = first_task[cell] + t; k < first_task[cell + 1]; k += NC)
#pragma unroll
    for (int c = 0; c < 9; ++c) acc[c] += red_w[(size_t)k * 9 + c];
#pragma unroll
  for (int c = 0; c < 9; ++c) sw[c][t] = acc[c];
  __syncthreads();
  for (int h = NC / 2; h > 0; h >>= 1) {
    if (t < h) {
#pragma unroll
      for (int c = 0; c < 9; ++c) sw[c][t] += sw[c][t + h];
    }
    __syncthreads();
  }
  if (t < 9) out[(size_t)cell * 9 + t] = sw[t][0];
}

constexpr double KAPPA = 9.648533212e-3;   // (eV/A)/amu in A/fs^2

__global__ __launch_bounds__(NT) void k_md_first(int n, double* __restrict__ x, double* __restrict__ y,
                                                 double* __restrict__ z, double* __restrict__ vx,
                                                 double* __restrict__ vy, double* __restrict__ vz,
                                                 const float* __restrict__ fx,
                                                 const float* __restrict__ fy,
                                                 const float* __restrict__ fz,
                                                 const int32_t* __restrict__ species, double h0,
                                                 double h1, double dt) {
  const int a = blockIdx.x * NT + threadIdx.x;
  if (a >= n) return;
  const double h = species[a] == 0 ? h0 : h1;    // dt/2 * KAPPA / m
  const double ux = vx[a] + h * (double)fx[a];
  const double uy = vy[a] + h * (double)fy[a];
  const double uz = vz[a] + h * (double)fz[a];
  vx[a] = ux;
  vy[a] = uy;
  vz[a] = uz;
  x[a] += dt * ux;
  y[a] += dt * uy;
  z[a] += dt * uz;
}

// The first half and drift of a step (as k_md_first) with, when the list stays, the
// displacement of each new position since the list build (as k_disp).
__global__ __launch_bounds__(NT) void k_md_first_drift(int n, double* __restrict__ x, double* __restrict__ y,
                                                       double* __restrict__ z, double* __restrict__ vx,
                                                       double* __restrict__ vy, double* __restrict__ vz,
                                                       const float* __restrict__ fx, const float* __restrict__ fy,
                                                       const float* __restrict__ fz,
                                                       const int32_t* __restrict__ species, double h0, double h1,
                                                       double dt, int disp, const double* __restrict__ xb,
                                                       const int* __restrict__ inv_perm, float4* __restrict__ dlt,
                                                       double lim2, int* __restrict__ status) {
  const int a = blockIdx.x * NT + threadIdx.x;
  if (a >= n) return;
  const double h = species[a] == 0 ? h0 : h1;    // dt/2 * KAPPA / m
  const double ux = vx[a] + h * (double)fx[a];
  const double uy = vy[a] + h * (double)fy[a];
  const double uz = vz[a] + h * (double)fz[a];
  vx[a] = ux;
  vy[a] = uy;
  vz[a] = uz;
  const double px = x[a] + dt * ux, py = y[a] + dt * uy, pz = z[a] + dt * uz;
  x[a] = px;
  y[a] = py;
  z[a] = pz;
  if (disp) store_displacement(a, n, px, py, pz, xb, inv_perm, dlt, lim2, status);
}

__global__ __launch_bounds__(NT) void k_md_second(int n, double* __restrict__ vx,
                                                  double* __restrict__ vy, double* __restrict__ vz,
                                                  const float* __restrict__ fx,
                                                  const float* __restrict__ fy,
                                                  const float* __restrict__ fz,
                                                  const int32_t* __restrict__ species, double h0,
                                                  double h1) {
  const int a = blockIdx.x * NT + threadIdx.x;
  if (a >= n) return;
  const double h = species[a] == 0 ? h0 : h1;
  vx[a] += h * (double)fx[a];
  vy[a] += h * (double)fy[a];
  vz[a] += h * (double)fz[a];
}

}  // namespace

namespace {
// per-cell reductions: energies and, with want_s, the largest sigma (red.sigma_max or a monitor)
void add_reduction(const flare_state* s, OutArgs& a, const Reduction& red) {
  a.want_e = red.e_struct != nullptr;
  a.want_s = red.sigma_max != nullptr || red.run_max != nullptr;
  if (!a.want_e && !a.want_s) return;
  a.task_groups = (int)s->tasks.size();
  a.cells = s->n_struct;
  a.tasks = s->d_tasks;
  a.bucket = s->bucket;
  a.e_int = s->e_int;
  a.v_int = s->v_int;
  a.red_e = s->red_e;
  a.red_s = s->red_s;
  a.first_task = s->d_first_task;
  a.e_struct = red.e_struct;
  a.sigma_max = red.sigma_max;
  a.thr = red.thr;
  a.run_max = red.run_max;
  a.over = red.over;
  a.status = s->d_status;
}
void add_outputs(const flare_state* s, OutArgs& a, const Outputs& out, const double* cell_scale) {
  a.n = s->n_atoms;
  a.atom_groups = (a.n + NT - 1) / NT;
  a.rows = a.n > 0 ? s->rows1 + s->rowsx : 0;
  a.row_groups = (a.rows + NT - 1) / NT;
  a.want_f = out.fx != nullptr;
  a.slice_base = s->slice_base;
  a.f_own = s->f_own;
  a.w_in = s->w_in;
  a.cnt_row = s->cnt_row;
  a.sid_row = s->sid_row;
  a.cell_scale = cell_scale;
  a.e_row = s->e_row;
  a.row_out = s->row_out;
  a.row_caller = s->row_caller;
  a.v_row = s->v_row;
  a.e_atom = out.e_atom;
  a.fx = out.fx;
  a.fy = out.fy;
  a.fz = out.fz;
  a.var_atom = out.var_atom;
  a.sigma_atom = out.sigma_atom;
}
void launch_outputs(const flare_state* s, const OutArgs& a) {
  if (a.row_groups + a.task_groups > 0)
    k_outputs_rows<<<a.row_groups + a.task_groups, NT, 0, s->stream>>>(a);
  const int cell_groups = (a.cells + NT / NC - 1) / (NT / NC);
  if (a.atom_groups + cell_groups > 0) k_outputs_atoms<<<a.atom_groups + cell_groups, NT, 0, s->stream>>>(a);
}
}  // namespace

void finalize_outputs(flare_state* s, const Outputs& out, const Reduction& red, const double* cell_scale) {
  OutArgs a{};
  add_outputs(s, a, out, cell_scale);
  add_reduction(s, a, red);
  launch_outputs(s, a);
}

void reduce_cells(flare_state* s, const Reduction& red) {
  OutArgs a{};
  add_reduction(s, a, red);
  launch_outputs(s, a);
}

void virial_cells(flare_state* s, double* virial_struct, double* red_w) {
  const int nt = (int)s->tasks.size();
  // as many threads as the longest task has atoms, up to 1,024: a task is one work-group, so a
  // cell of a few thousand atoms has few of them (7.7 k atoms: 46 us with 256 threads, 30 with
  // 1,024; 100 cells of 800: 28 and 14), and a batch of small cells has many nearly empty ones
  // (20,000 cells of 4: 181 us with 1,024 threads, 72 with 256, 46 with 64; 500 cells of 100:
  // 12, 12 and 18)
  const int nv = s->longest_task <= 64 ? 64 : s->longest_task <= 256 ? 256 : 1024;
  auto tasks = nv == 64 ? k_virial_tasks<64> : nv == 256 ? k_virial_tasks<256> : k_virial_tasks<1024>;
  if (nt > 0)
    tasks<<<nt, nv, 0, s->stream>>>(s->d_tasks, s->bucket, s->row_of, s->rows1, s->slice_base, s->geom, s->w_in,
                                    s->nl_cnt, red_w);
  if (s->n_struct > 0)
    k_virial_cells<<<s->n_struct, NC, 0, s->stream>>>(red_w, s->d_first_task, virial_struct);
}

void md_first(flare_state* s, double* x, double* y, double* z, double* vx, double* vy, double* vz,
              const float* fx, const float* fy, const float* fz, const int32_t* species,
              double inv_m0, double inv_m1, double dt) {
  const int n = s->n_atoms;
  if (n == 0) return;
  const double h0 = 0.5 * dt * KAPPA * inv_m0, h1 = 0.5 * dt * KAPPA * inv_m1;
  k_md_first<<<(n + NT - 1) / NT, NT, 0, s->stream>>>(n, x, y, z, vx, vy, vz, fx, fy, fz, species, h0, h1, dt);
}

void md_first_drift(flare_state* s, double* x, double* y, double* z, double* vx, double* vy, double* vz,
                    const float* fx, const float* fy, const float* fz, const int32_t* species, double inv_m0,
                    double inv_m1, double dt, bool displacements) {
  const int n = s->n_atoms;
  if (n == 0) return;
  const double h0 = 0.5 * dt * KAPPA * inv_m0, h1 = 0.5 * dt * KAPPA * inv_m1;
  const double lim = 0.5 * s->skin;
  k_md_first_drift<<<(n + NT - 1) / NT, NT, 0, s->stream>>>(n, x, y, z, vx, vy, vz, fx, fy, fz, species, h0, h1,
                                                            dt, displacements ? 1 : 0, s->xb, s->inv_perm, s->dlt,
                                                            lim * lim, s->d_status);
}

void outputs_second_half(flare_state* s, const Outputs& out, const Reduction& red, double* vx, double* vy, double* vz,
                         const int32_t* species, double inv_m0, double inv_m1, double dt) {
  OutArgs a{};
  add_outputs(s, a, out, nullptr);
  add_reduction(s, a, red);
  a.vx = vx;
  a.vy = vy;
  a.vz = vz;
  a.species = species;
  a.h0 = 0.5 * dt * KAPPA * inv_m0;
  a.h1 = 0.5 * dt * KAPPA * inv_m1;
  launch_outputs(s, a);
}

void md_second(flare_state* s, double* vx, double* vy, double* vz, const float* fx, const float* fy,
               const float* fz, const int32_t* species, double inv_m0, double inv_m1, double dt) {
  const int n = s->n_atoms;
  if (n == 0) return;
  const double h0 = 0.5 * dt * KAPPA * inv_m0, h1 = 0.5 * dt * KAPPA * inv_m1;
  k_md_second<<<(n + NT - 1) / NT, NT, 0, s->stream>>>(n, vx, vy, vz, fx, fy, fz, species, h0, h1);
}

}  // namespace flare
