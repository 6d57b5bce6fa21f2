// Device-wide exclusive prefix sums of int32 counts (bin counts, pair counts, bucket counts,
// slice lengths), out[0..n-1] and the total out[n]: up to 16,384 elements in one launch of a
// single work-group, more in two, the totals of 1024-element blocks, then each block's scan
// from the sum of the totals before it (at most a few thousand, read by every block). Two
// arrays can share the launches (scan_exclusive2). Deterministic (integer).
#include "common.h"

namespace flare {

namespace {

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_PER_THREAD = 4;
constexpr int SCAN_BLOCK = SCAN_THREADS * SCAN_PER_THREAD;   // 1024 elements per block
constexpr int ONE_THREADS = 1024;
constexpr int ONE_MAX = 16 * ONE_THREADS;                    // elements of the one-launch form

template <class T>
__device__ inline T wave_incl_scan(T v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const T t = __shfl_up(v, d, 64);
    if (lane >= d) v += t;
  }
  return v;
}

// One array of a scan: its blocks are [block0, block0 + nb) of the launch, its block totals
// start at sums. status: the flag is raised there when the total passes 2^31 - 1.
struct ScanJob {
  const int* in;
  int* out;
  int n;
  int nb;
  long long* sums;
  int* status;
  int flag;
};

// Phase 1: the total of every 1024-element block.
__device__ void block_sums(const ScanJob& j, int block) {
  __shared__ long long wsum[SCAN_THREADS / 64];
  const long long base = (long long)block * SCAN_BLOCK + threadIdx.x * SCAN_PER_THREAD;
  long long tot = 0;
#pragma unroll
  for (int k = 0; k < SCAN_PER_THREAD; ++k) tot += base + k < j.n ? j.in[base + k] : 0;
  const long long incl = wave_incl_scan(tot);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long t = 0;
    for (int k = 0; k < SCAN_THREADS / 64; ++k) t += wsum[k];
    j.sums[block] = t;
  }
}

// Phase 2: every block adds up the totals of the blocks before it, scans its own elements
// from there and writes them; the block holding element n - 1 also writes the total out[n].
__device__ void scan_block(const ScanJob& j, int block) {
  __shared__ long long wsum[SCAN_THREADS / 64];
  __shared__ long long pre_s;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  long long pre = 0;
  for (int k = threadIdx.x; k < block; k += SCAN_THREADS) pre += j.sums[k];
  pre = wave_incl_scan(pre);
  if (lane == 63) wsum[w] = pre;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long t = 0;
    for (int k = 0; k < SCAN_THREADS / 64; ++k) t += wsum[k];
    pre_s = t;
  }
  __syncthreads();
  const long long block_pre = pre_s;
  const long long base = (long long)block * SCAN_BLOCK + threadIdx.x * SCAN_PER_THREAD;
  int v[SCAN_PER_THREAD];
  long long tot = 0;
#pragma unroll
  for (int k = 0; k < SCAN_PER_THREAD; ++k) {
    v[k] = base + k < j.n ? j.in[base + k] : 0;
    tot += v[k];
  }
  const long long incl = wave_incl_scan(tot);
  __syncthreads();                       // wsum is reused
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  long long woff = 0;
  for (int k = 0; k < w; ++k) woff += wsum[k];
  long long run = block_pre + woff + incl - tot;
#pragma unroll
  for (int k = 0; k < SCAN_PER_THREAD; ++k) {
    if (base + k < j.n) j.out[base + k] = (int)run;
    run += v[k];
  }
  // the total: written by the thread that holds element n - 1 (its running sum has passed
  // it; the elements past n counted as zeros)
  if (base <= (long long)j.n - 1 && (long long)j.n - 1 < base + SCAN_PER_THREAD) {
    j.out[j.n] = (int)run;
    if (j.status && run > 0x7fffffffLL) atomicOr(j.status, j.flag);
  }
}

__global__ __launch_bounds__(SCAN_THREADS) void k_block_sums(ScanJob a, ScanJob b) {
  if ((int)blockIdx.x < a.nb) block_sums(a, blockIdx.x);
  else block_sums(b, blockIdx.x - a.nb);
}
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_blocks(ScanJob a, ScanJob b) {
  if ((int)blockIdx.x < a.nb) scan_block(a, blockIdx.x);
  else scan_block(b, blockIdx.x - a.nb);
}

// A work-group per array of at most ONE_MAX elements, 16 consecutive ones a thread.
__global__ __launch_bounds__(ONE_THREADS) void k_scan_one(ScanJob a, ScanJob b) {
  const ScanJob j = blockIdx.x == 0 ? a : b;
  __shared__ long long wsum[ONE_THREADS / 64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int per = (j.n + ONE_THREADS - 1) / ONE_THREADS;
  const int base = threadIdx.x * per;
  long long tot = 0;
  for (int k = 0; k < per; ++k) tot += base + k < j.n ? j.in[base + k] : 0;
  const long long incl = wave_incl_scan(tot);
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  long long run = incl - tot;
  for (int k = 0; k < w; ++k) run += wsum[k];
  for (int k = 0; k < per; ++k)
    if (base + k < j.n) {
      j.out[base + k] = (int)run;
      run += j.in[base + k];
    }
  if (threadIdx.x == ONE_THREADS - 1) {
    long long t = 0;
    for (int k = 0; k < ONE_THREADS / 64; ++k) t += wsum[k];
    j.out[j.n] = (int)t;
    if (j.status && t > 0x7fffffffLL) atomicOr(j.status, j.flag);
  }
}

int nblocks(long long n) { return (int)((n + SCAN_BLOCK - 1) / SCAN_BLOCK); }

void launch_scan(ScanJob a, ScanJob b, int jobs, hipStream_t st) {
  if (a.n <= ONE_MAX && (jobs < 2 || b.n <= ONE_MAX)) {
    k_scan_one<<<jobs, ONE_THREADS, 0, st>>>(a, b);
    return;
  }
  // an empty array still gets one block, which writes its total
  if (a.n == 0 || (jobs > 1 && b.n == 0)) {
    launch_scan(a, a, 1, st);
    if (jobs > 1) launch_scan(b, b, 1, st);
    return;
  }
  k_block_sums<<<a.nb + b.nb, SCAN_THREADS, 0, st>>>(a, b);
  k_scan_blocks<<<a.nb + b.nb, SCAN_THREADS, 0, st>>>(a, b);
}

}  // namespace

size_t scan_scratch_ints(long long n) { return 2 * ((size_t)nblocks(n) + 64); }

void scan_exclusive(const int* in, int* out, int n, int* scratch, hipStream_t st) {
  const ScanJob a{in, out, n, nblocks(n), reinterpret_cast<long long*>(scratch), nullptr, 0};
  launch_scan(a, ScanJob{}, 1, st);
}

void scan_exclusive2(const int* in0, int* out0, int n0, const int* in1, int* out1, int n1, int* scratch, int* status,
                     int flag, hipStream_t st) {
  long long* sums = reinterpret_cast<long long*>(scratch);
  const ScanJob a{in0, out0, n0, nblocks(n0), sums, status, flag};
  const ScanJob b{in1, out1, n1, nblocks(n1), sums + nblocks(n0) + 1, nullptr, 0};
  launch_scan(a, b, 2, st);
}

}  // namespace flare
