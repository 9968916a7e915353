// Counting sort of the particle arrays by element (active particles first,
// in element order; inactive ones at the end).  Histogram with atomics, an
// exclusive scan over the E+1 buckets of particles and of element tasks, which
// clears the histogram for the next sort, then a scatter of every SoA field, in
// which the first particle of each task writes it (a thread of the scan would
// write the tasks of its buckets one after the other: 1e6 particles in 8
// elements 1640 us a sort instead of 267, in 16^3 103 instead of 88).  The tasks
// are cut both ways, 32 and 64 particles: the steps that follow a sort may need
// either (precision, extra forces, the source), one after the other or in a
// captured graph.
// Launches of a few microseconds each are what a sort of few particles costs:
// clear, histogram, two three-launch scans, task count, task fill and scatter
// were 11 of them (46 us for 1e4 particles); one scan of bucket starts and task
// starts together leaves three, or four beyond kScanTile buckets.
#include "fp_launch.h"

namespace fp {

// rank of each particle within its bucket.  The particles are mostly in
// element order already (sorted at the last step, few crossings since), so
// neighbouring lanes share keys: one atomic per run of equal keys within a
// wavefront instead of one per particle (atomics on one address serialise)
__global__ __launch_bounds__(256) void k_sort_hist(const int8_t* __restrict__ status,
                                                   const int32_t* __restrict__ elem, int64_t n, int E,
                                                   int32_t* count, int32_t* rank) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const bool valid = p < n;
  const int key = valid ? (status[p] == ACTIVE ? elem[p] : E) : -1;
  const int prev = __shfl_up(key, 1, 64);
  const bool head = valid && (lane == 0 || prev != key);
  const unsigned long long heads = __ballot(head);
  const int nvalid = (int)__popcll(__ballot(valid));   // the valid lanes are a prefix
  int base = 0;
  if (head) {
    const unsigned long long above = lane == 63 ? 0ull : heads >> (lane + 1);
    const int next = above ? lane + 1 + __builtin_ctzll(above) : nvalid;
    base = atomicAdd(count + key, next - lane);
  }
  // the head of this lane's run: the highest head at or below the lane
  const unsigned long long upto = heads & (lane == 63 ? ~0ull : ((1ull << (lane + 1)) - 1ull));
  const int start = upto ? 63 - __builtin_clzll(upto) : 0;
  const int b = __shfl(base, start, 64);
  if (valid) rank[p] = b + (lane - start);
}

// exclusive scan of 1024-entry tiles (256 threads x 4), tile totals to sums
__global__ __launch_bounds__(256) void k_scan_tiles(const int32_t* in, int32_t* out, int64_t n, int32_t* sums) {
  __shared__ int32_t sh[256];
  int64_t base = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
  int32_t v[4], s = 0;
  for (int k = 0; k < 4; ++k) {
    v[k] = (base + k < n) ? in[base + k] : 0;
    s += v[k];
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {
    int32_t t = (threadIdx.x >= (unsigned)off) ? sh[threadIdx.x - off] : 0;
    __syncthreads();
    sh[threadIdx.x] += t;
    __syncthreads();
  }
  int32_t run = sh[threadIdx.x] - s;
  for (int k = 0; k < 4; ++k) {
    if (base + k < n) out[base + k] = run;
    run += v[k];
  }
  if (threadIdx.x == 255) sums[blockIdx.x] = sh[255];
}

// exclusive scan of the tile totals by one block (loops over chunks of 1024)
__global__ __launch_bounds__(256) void k_scan_sums(int32_t* sums, int64_t nt) {
  __shared__ int32_t sh[256];
  int32_t carry = 0;
  for (int64_t c0 = 0; c0 < nt; c0 += 1024) {
    int64_t base = c0 + threadIdx.x * 4;
    int32_t v[4], s = 0;
    for (int k = 0; k < 4; ++k) {
      v[k] = (base + k < nt) ? sums[base + k] : 0;
      s += v[k];
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
      int32_t t = (threadIdx.x >= (unsigned)off) ? sh[threadIdx.x - off] : 0;
      __syncthreads();
      sh[threadIdx.x] += t;
      __syncthreads();
    }
    int32_t run = carry + sh[threadIdx.x] - s;
    for (int k = 0; k < 4; ++k) {
      if (base + k < nt) sums[base + k] = run;
      run += v[k];
    }
    int32_t tot = sh[255];
    __syncthreads();
    carry += tot;
  }
}

__global__ void k_scan_add(int32_t* out, int64_t n, const int32_t* sums) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] += sums[i / 1024];
}

__global__ __launch_bounds__(256) void k_sort_scatter(Particles S, Particles D, int64_t n, int E,
                                                      const int32_t* __restrict__ start,
                                                      const int32_t* __restrict__ rank,
                                                      const int2* __restrict__ tstart, Task* __restrict__ tasks32,
                                                      Task* __restrict__ tasks64) {
  int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  int8_t st = S.status[p];
  int32_t e = S.elem[p];
  int key = st == ACTIVE ? e : E;
  const int r = rank[p];
  int64_t q = (int64_t)start[key] + r;
  if (key < E && r % 32 == 0) {
    const int2 t = tstart[key];
    const int left = start[key + 1] - (int32_t)q;
    tasks32[t.x + r / 32] = Task{key, (int32_t)q, min(32, left), 0};
    if (r % 64 == 0) tasks64[t.y + r / 64] = Task{key, (int32_t)q, min(64, left), 0};
  }
  const int64_t cs = S.cap, cd = D.cap;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    D.x[k * cd + q] = S.x[k * cs + p];
    D.v[k * cd + q] = S.v[k * cs + p];
    D.kx[k * cd + q] = S.kx[k * cs + p];
    D.kv[k * cd + q] = S.kv[k * cs + p];
    D.xi[k * cd + q] = S.xi[k * cs + p];
  }
  D.d[q] = S.d[p];
  D.elem[q] = e;
  D.hits[q] = S.hits[p];
  D.id[q] = S.id[p];
  D.status[q] = st;
}

hipError_t scan_i32(const int32_t* in, int32_t* out, int64_t n, int32_t* sums, hipStream_t s) {
  int64_t nt = (n + 1023) / 1024;
  k_scan_tiles<<<dim3((unsigned)nt), 256, 0, s>>>(in, out, n, sums);
  k_scan_sums<<<1, 256, 0, s>>>(sums, nt);
  k_scan_add<<<dim3((unsigned)((n + 255) / 256)), 256, 0, s>>>(out, n, sums);
  return hipGetLastError();
}

constexpr int kScanPer = 16, kScanTile = 256 * kScanPer;   // buckets per thread and per workgroup

// what the scan adds up: particles, tasks of 32 and tasks of 64
struct SortSum { int p, t32, t64; };

__device__ __forceinline__ SortSum operator+(SortSum a, SortSum b) { return {a.p + b.p, a.t32 + b.t32, a.t64 + b.t64}; }

// bucket e of c particles (bucket E, the inactive particles, has no tasks)
__device__ __forceinline__ SortSum bucket_sum(int c, bool element) {
  return {c, element ? (c + 31) / 32 : 0, element ? (c + 63) / 64 : 0};
}

// exclusive prefix over the workgroup's 256 threads, and the sum
__device__ __forceinline__ SortSum block_scan(SortSum a, SortSum* total) {
  __shared__ SortSum sums[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  SortSum x = a;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const SortSum u{__shfl_up(x.p, o, 64), __shfl_up(x.t32, o, 64), __shfl_up(x.t64, o, 64)};
    if (lane >= o) x = x + u;
  }
  if (lane == 63) sums[wave] = x;
  __syncthreads();
  SortSum before{0, 0, 0};
  *total = before;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (w < wave) before = before + sums[w];
    *total = *total + sums[w];
  }
  __syncthreads();
  return {before.p + x.p - a.p, before.t32 + x.t32 - a.t32, before.t64 + x.t64 - a.t64};
}

// sums of each tile of buckets
__global__ __launch_bounds__(256) void k_sort_sums(const int32_t* __restrict__ count, int E, SortSum* sums) {
  const int64_t b0 = (int64_t)blockIdx.x * kScanTile;
  SortSum a{0, 0, 0}, total;
  for (int k = 0; k < kScanPer; ++k) {
    const int64_t e = b0 + k * 256 + threadIdx.x;
    if (e <= E) a = a + bucket_sum(count[e], e < E);
  }
  block_scan(a, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// starts of the buckets' particles and of their tasks of either size, and the
// numbers of tasks; the histogram is cleared.  sums: every tile's sums (the
// workgroup adds those before its own: a few hundred values for the largest
// meshes).
__global__ __launch_bounds__(256) void k_sort_scan(int32_t* __restrict__ count, int32_t* __restrict__ start, int E,
                                                   const SortSum* __restrict__ sums, int2* __restrict__ tstart,
                                                   int32_t* ntask) {
  SortSum before{0, 0, 0}, total;
  if (blockIdx.x > 0) {
    SortSum a{0, 0, 0};
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += 256) a = a + sums[t];
    block_scan(a, &before);
  }
  const int64_t e0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
  int c[kScanPer];
  SortSum a{0, 0, 0};
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    c[k] = e0 + k <= E ? count[e0 + k] : 0;
    a = a + bucket_sum(c[k], e0 + k < E);
  }
  a = before + block_scan(a, &total);
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    const int64_t e = e0 + k;
    if (e > E) break;
    start[e] = a.p;
    count[e] = 0;
    if (e < E) {
      tstart[e] = make_int2(a.t32, a.t64);
    } else {
      ntask[0] = a.t32;
      ntask[1] = a.t64;
    }
    a = a + bucket_sum(c[k], e < E);
  }
}

hipError_t launch_sort(const Particles& src, const Particles& dst, int64_t n, int E, int32_t* count, int32_t* start,
                       int32_t* rank, int32_t* sums, int32_t* tstart, void* tasks32, void* tasks64, int32_t* ntask,
                       hipStream_t s) {
  if (n == 0) return hipSuccess;
  const dim3 g((unsigned)((n + 255) / 256)), tiles((unsigned)((E + kScanTile) / kScanTile));   // E + 1 buckets
  k_sort_hist<<<g, 256, 0, s>>>(src.status, src.elem, n, E, count, rank);
  if (tiles.x > 1) k_sort_sums<<<tiles, 256, 0, s>>>(count, E, (SortSum*)sums);
  k_sort_scan<<<tiles, 256, 0, s>>>(count, start, E, (const SortSum*)sums, (int2*)tstart, ntask);
  k_sort_scatter<<<g, 256, 0, s>>>(src, dst, n, E, start, rank, (const int2*)tstart, (Task*)tasks32, (Task*)tasks64);
  return hipGetLastError();
}

__global__ void k_clear_i32(int32_t* a, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = 0;
}

hipError_t launch_clear_i32(int32_t* a, int64_t n, hipStream_t s) {
  k_clear_i32<<<dim3((unsigned)((n + 255) / 256)), 256, 0, s>>>(a, n);
  return hipGetLastError();
}

// the first n particles of S to the same rows of D (a caller-owned block)
__global__ __launch_bounds__(256) void k_copy_particles(Particles S, Particles D, int64_t n) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const int64_t cs = S.cap, cd = D.cap;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    D.x[k * cd + p] = S.x[k * cs + p];
    D.v[k * cd + p] = S.v[k * cs + p];
    D.kx[k * cd + p] = S.kx[k * cs + p];
    D.kv[k * cd + p] = S.kv[k * cs + p];
    D.xi[k * cd + p] = S.xi[k * cs + p];
  }
  D.d[p] = S.d[p];
  D.elem[p] = S.elem[p];
  D.hits[p] = S.hits[p];
  D.id[p] = S.id[p];
  D.status[p] = S.status[p];
}

hipError_t launch_copy_particles(const Particles& S, const Particles& D, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_copy_particles<<<dim3((unsigned)((n + 255) / 256)), 256, 0, s>>>(S, D, n);
  return hipGetLastError();
}

size_t task_bytes() { return sizeof(Task); }

}  // namespace fp
