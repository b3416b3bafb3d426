// Periodic cell sort: a stable counting sort of one species by cell index
// j = clamp(floor(x / dx), 0, N_x - 2), which keeps the particles of a tile in
// a few neighbouring cells so the particle kernel's deposit flush and its
// field gathers stay local. Stable, so the result is a pure function of the
// input order. Three launches, each for both species and all discharges due:
//   count   per-chunk key histograms (LDS), written key-major
//   scan    a wave per key, or as many lanes of one as there are chunks:
//           exclusive sums of the key's counts over the chunks, and its total
//   scatter the keys' bases from their totals, then 2048 particles of a chunk
//           at a time: each wave ranks its 256 in registers (lanes of equal
//           keys by ballots), the waves' counts are summed per key, and
//           everything goes to its place.
// A sort step is latency, not bandwidth, at most sizes: it was five launches
// per species, and the scatter walked a chunk 256 particles at a time with a
// barrier per wave and two dependent loads exposed in each. Kernel times of both
// species' sorts, 5 thousand particles of each on 64 cells: 49 -> 14 us; 400
// thousand on 512 cells: 78 -> 25 us; 16 discharges of 300 thousand on 64: 222
// -> 190 us.
#include "pic_internal.h"

namespace pic {

constexpr int kSortThreads = 256;
constexpr int kScatThreads = 512;
constexpr int kScatWaves = kScatThreads / kWave;
constexpr int kScatPer = 4;  // particles of a lane
constexpr int kScatChunk = kScatThreads * kScatPer;
static_assert(kMaxSortBlocks % kWave == 0, "k_sort_scan reads whole rounds of a wave");

__device__ __forceinline__ void chunk_range(int64_t n, int nblocks, int b, int64_t& lo,
                                            int64_t& hi) {
  const int64_t chunk = (n + nblocks - 1) / nblocks;
  lo = (int64_t)b * chunk;
  hi = lo + chunk;
  if (hi > n) hi = n;
  if (lo > n) lo = n;
}

// Chunk b of a's input: per-key counts, written key-major.
__device__ __forceinline__ void sort_count_block(const SortArgs& a, int b, uint32_t* sh) {
  const int nkeys = a.nx - 1;
  for (int k = threadIdx.x; k < nkeys; k += kSortThreads) sh[k] = 0u;
  __syncthreads();
  int64_t lo, hi;
  chunk_range(min(*a.count, a.cap), a.nblocks, b, lo, hi);
  for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += 8 * kSortThreads) {
    double x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = a.sx[min(i0 + q * kSortThreads, hi - 1)];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (i0 + q * kSortThreads < hi) atomicAdd(&sh[cell_key(x[q], a.inv_dx, a.nx)], 1u);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < nkeys; k += kSortThreads)
    a.cnt[(size_t)k * a.nblocks + b] = sh[k];
}

// Keys of `lanes` lanes each (a power of two, at least the chunks): as
// sort_scan_key, lane t of all.
__device__ __forceinline__ void sort_scan_keys(const SortArgs& a, int t, int lanes) {
  const int k = t / lanes, i = t & (lanes - 1);
  const bool in = k < a.nx - 1 && i < a.nblocks;
  uint32_t* row = a.cnt + (size_t)k * a.nblocks;
  const uint32_t v = in ? row[i] : 0u;
  uint32_t inc = v;
  for (int d = 1; d < lanes; d <<= 1) {
    const uint32_t w = (uint32_t)__shfl_up((int)inc, d, lanes);
    if (i >= d) inc += w;
  }
  if (in) row[i] = inc - v;
  if (i == lanes - 1 && k < a.nx - 1) a.tot[k] = inc;
}

// Key k (one wave): its counts become the counts of the chunks before.
__device__ __forceinline__ void sort_scan_key(const SortArgs& a, int k) {
  constexpr int kRounds = kMaxSortBlocks / kWave;
  const int lane = threadIdx.x & (kWave - 1);
  uint32_t* row = a.cnt + (size_t)k * a.nblocks;
  uint32_t v[kRounds];
#pragma unroll
  for (int q = 0; q < kRounds; ++q) {
    const int i = q * kWave + lane;
    v[q] = i < a.nblocks ? row[i] : 0u;
  }
  uint32_t run = 0u;
#pragma unroll
  for (int q = 0; q < kRounds; ++q) {
    if (q * kWave >= a.nblocks) break;
    const uint32_t inc = wave_incl_scan<unsigned int>(v[q]);
    const int i = q * kWave + lane;
    if (i < a.nblocks) row[i] = run + inc - v[q];
    run += (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
  }
  if (lane == 0) a.tot[k] = run;
}

static size_t scatter_lds(int nx) { return (size_t)(nx - 1) * (4 + 2 * (kScatWaves + 1)); }

// LDS: a 32-bit output position per key, then a 16-bit count per key of each
// wave (then of the waves before it) and of all of them.
__device__ __forceinline__ void sort_scatter_block(const SortArgs& a, int b, uint32_t* off) {
  __shared__ uint32_t s_w[kScatWaves];
  const int nkeys = a.nx - 1;
  uint16_t* cw = reinterpret_cast<uint16_t*>(off + nkeys);
  const int tid = threadIdx.x;
  const int wave = tid / kWave;
  const int lane = tid & (kWave - 1);
  uint16_t* mine = cw + (size_t)wave * nkeys;
  uint16_t* all = cw + (size_t)kScatWaves * nkeys;
  {
    // first position of each key, and of this chunk's particles in it
    const int per = (nkeys + kScatThreads - 1) / kScatThreads;
    const int k0 = min(tid * per, nkeys), k1 = min(k0 + per, nkeys);
    uint32_t sum = 0u;
    for (int k = k0; k < k1; ++k) sum += a.tot[k];
    const uint32_t inc = wave_incl_scan<unsigned int>(sum);
    if (lane == kWave - 1) s_w[wave] = inc;
    __syncthreads();
    uint32_t base = inc - sum;
    for (int w = 0; w < wave; ++w) base += s_w[w];
    for (int k = k0; k < k1; ++k) {
      off[k] = base + a.cnt[(size_t)k * a.nblocks + b];
      base += a.tot[k];
    }
  }
  int64_t lo, hi;
  const int64_t n = min(uniform64(*a.count), a.cap);
  // the rebuilt pool holds exactly the n sorted slots
  if (b == 0 && tid == 0) *a.pool_n = n;
  chunk_range(n, a.nblocks, b, lo, hi);
  lo = uniform64(lo);
  hi = uniform64(hi);
  const uint64_t lt = (1ull << lane) - 1ull;
  const int bits = 32 - __builtin_clz((unsigned)(nkeys - 1) | 1u);
  for (int64_t b0 = lo; b0 < hi; b0 += kScatChunk) {
    double x[kScatPer], vx[kScatPer];
    double vy[kScatPer], vz[kScatPer];
    uint32_t id[kScatPer];
    const int64_t i0 = b0 + wave * (kWave * kScatPer) + lane;
#pragma unroll
    for (int r = 0; r < kScatPer; ++r) {
      const int64_t i = min(i0 + r * kWave, hi - 1);
      id[r] = a.sid[i];
      x[r] = a.sx[i];
      vx[r] = a.svx[i];
    }
#pragma unroll
    for (int r = 0; r < kScatPer; ++r) {
      const double2 v = a.spv[id[r]];
      vy[r] = v.x;
      vz[r] = v.y;
    }
    for (int k = lane; k < nkeys; k += kWave) mine[k] = 0;
    int key[kScatPer];
    uint32_t rank[kScatPer];
#pragma unroll
    for (int r = 0; r < kScatPer; ++r) {
      const bool valid = i0 + r * kWave < hi;
      key[r] = cell_key(x[r], a.inv_dx, a.nx);
      // lanes of this wave holding the same key
      uint64_t mask = __ballot(valid);
      for (int bit = 0; bit < bits; ++bit) {
        const bool on = (key[r] >> bit) & 1;
        const uint64_t bm = __ballot(valid && on);
        mask &= on ? bm : ~bm;
      }
      // the wave's counts so far: read, then raised by the first lane of each
      // key (LDS operations of a wave are performed in order)
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const uint32_t before = mine[key[r]];
      rank[r] = before + (uint32_t)__popcll(mask & lt);
      if (valid && (mask & lt) == 0) mine[key[r]] = (uint16_t)(before + (uint32_t)__popcll(mask));
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __syncthreads();
    for (int k = tid; k < nkeys; k += kScatThreads) {
      uint32_t run = 0u;
#pragma unroll
      for (int w = 0; w < kScatWaves; ++w) {
        const uint32_t c = cw[(size_t)w * nkeys + k];
        cw[(size_t)w * nkeys + k] = (uint16_t)run;
        run += c;
      }
      all[k] = (uint16_t)run;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kScatPer; ++r)
      if (i0 + r * kWave < hi) {
        // the sorted slot's pool entry is the slot itself
        const uint32_t dest = off[key[r]] + mine[key[r]] + rank[r];
        a.dx[dest] = x[r];
        a.dvx[dest] = vx[r];
        a.did[dest] = dest;
        a.dpv[dest] = make_double2(vy[r], vz[r]);
      }
    if (b0 + kScatChunk < hi) {
      __syncthreads();
      for (int k = tid; k < nkeys; k += kScatThreads) off[k] += all[k];
    }
  }
}

// Both species of one discharge, a row of the grid each.
struct SortPair {
  SortArgs a[2];
};

__global__ __launch_bounds__(kSortThreads) void k_sort_count(SortPair p) {
  extern __shared__ uint32_t sh[];
  sort_count_block(p.a[blockIdx.y], blockIdx.x, sh);
}

// workgroup b of a's scan
__device__ __forceinline__ void sort_scan_block(const SortArgs& a, int b, int lanes) {
  if (lanes < kWave) {
    sort_scan_keys(a, b * kSortThreads + (int)threadIdx.x, lanes);
  } else {
    const int k = b * (kSortThreads / kWave) + threadIdx.x / kWave;
    if (k < a.nx - 1) sort_scan_key(a, k);
  }
}

__global__ __launch_bounds__(kSortThreads) void k_sort_scan(SortPair p, int lanes) {
  sort_scan_block(p.a[blockIdx.y], blockIdx.x, lanes);
}

__global__ __launch_bounds__(kScatThreads) void k_sort_scatter(SortPair p) {
  extern __shared__ uint32_t off[];
  sort_scatter_block(p.a[blockIdx.y], blockIdx.x, off);
}

// ---------------------------------------------------------------------------
// Batched sorts: n discharges (their electrons at e, their ions at i, each
// with its own counters) in one launch per kernel, a row of the grid per
// species. Count and scatter lay the discharges' chunk blocks end to end; the
// scan takes the blocks of the largest grid for each.

// The job of this workgroup among jobs whose block counts are nb(j), and
// the workgroup's block within it.
template <int THREADS>
__device__ __forceinline__ void job_block(const SortArgs* __restrict__ args, int n, int& job,
                                          int& b) {
  __shared__ int64_t s_bs[kMaxBatch + 1];
  __shared__ int64_t s_w[THREADS / kWave];
  block_exclusive<THREADS>(threadIdx.x < (unsigned)n ? args[threadIdx.x].nblocks : 0, n, s_bs, s_w);
  const int64_t g = blockIdx.x;
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (s_bs[mid] <= g) lo = mid;
    else hi = mid - 1;
  }
  job = uniform32(lo);
  b = uniform32((int)(g - s_bs[lo]));
}

__global__ __launch_bounds__(kSortThreads) void k_sort_count_b(const SortArgs* __restrict__ e,
                                                                const SortArgs* __restrict__ i,
                                                                int n) {
  extern __shared__ uint32_t sh[];
  const SortArgs* args = blockIdx.y ? i : e;
  int job, b;
  job_block<kSortThreads>(args, n, job, b);
  sort_count_block(args[job], b, sh);
}

__global__ __launch_bounds__(kSortThreads) void k_sort_scan_b(const SortArgs* __restrict__ e,
                                                               const SortArgs* __restrict__ i,
                                                               int blocks, int lanes) {
  sort_scan_block((blockIdx.y ? i : e)[blockIdx.x / blocks], blockIdx.x % blocks, lanes);
}

__global__ __launch_bounds__(kScatThreads) void k_sort_scatter_b(const SortArgs* __restrict__ e,
                                                                  const SortArgs* __restrict__ i,
                                                                  int n) {
  extern __shared__ uint32_t off[];
  const SortArgs* args = blockIdx.y ? i : e;
  int job, b;
  job_block<kScatThreads>(args, n, job, b);
  sort_scatter_block(args[job], b, off);
}

// A chunk costs every kernel a pass over the cells (the counts of a cell lie a
// chunk apart), so a launch takes about as many chunks as scatter workgroups
// are resident (the LDS of a wide grid leaves one per CU, 2048 points three),
// of at least the particles one takes at a time. A discharge alone has two such
// rounds, which overlap, where several workgroups fit, and where they do a
// chunk is no longer than 16384 (16 million of both on 2048 cells: 392 us with
// 20800 each, 345). Kernel times of the sorts of both species, with chunks of
// capacity / 4096 for every discharge and a wave per cell's scan -> now:
//   400 thousand of each, 2048 / 4096 cells        52 / 112 -> 37 / 50 us
//   8 million, 2048 / 4096                        345 / 450 -> 344 / 400
//   16 discharges of 300 thousand, 1200 / 4096   394 / 1347 -> 213 / 275
//   64 of 100 thousand, 1200 / 4096              551 / 1852 -> 288 / 332
//   256 of 1000, 512 / 4096                        60 / 363 -> 25 / 54
SortShape sort_chunks(SortArgs* e, SortArgs* i, int n, int nx_max, int num_cu) {
  constexpr int kFit = 2048 / kScatThreads;
  const int lds = (int)(160 * 1024 / (scatter_lds(nx_max) + 4096));
  const int fit = lds < 1 ? 1 : lds > kFit ? kFit : lds;
  int64_t all = 0;
  for (int k = 0; k < n; ++k) all += e[k].hint + i[k].hint;
  int64_t per = all / ((int64_t)num_cu * fit * (fit > 1 && n == 1 ? 2 : 1));
  if (fit > 1 && per > 16384) per = 16384;
  if (per < kScatChunk) per = kScatChunk;
  SortShape c{0, 1};
  for (int k = 0; k < n; ++k) {
    const int64_t most = e[k].hint > i[k].hint ? e[k].hint : i[k].hint;
    const int64_t want = (most + per - 1) / per;
    const int nb = want < 1 ? 1 : want > e[k].nblocks ? e[k].nblocks : (int)want;
    e[k].nblocks = i[k].nblocks = nb;
    c.blocks += nb;
    while (c.lanes < nb && c.lanes < kWave) c.lanes *= 2;
  }
  return c;
}

static int scan_blocks(int nx, int lanes) {
  return (int)(((int64_t)(nx - 1) * lanes + kSortThreads - 1) / kSortThreads);
}

hipError_t launch_batch_sort(const SortArgs* e, const SortArgs* i, int n, const SortShape& c,
                             int nx_max, hipStream_t s) {
  if (n < 1 || n > kMaxBatch || c.blocks < 1 || nx_max < 3) return hipErrorInvalidValue;
  const int sb = scan_blocks(nx_max, c.lanes);
  hipLaunchKernelGGL(k_sort_count_b, dim3((unsigned)c.blocks, 2), dim3(kSortThreads),
                     (size_t)(nx_max - 1) * 4, s, e, i, n);
  hipLaunchKernelGGL(k_sort_scan_b, dim3((unsigned)(n * sb), 2), dim3(kSortThreads), 0, s, e, i, sb,
                     c.lanes);
  hipLaunchKernelGGL(k_sort_scatter_b, dim3((unsigned)c.blocks, 2), dim3(kScatThreads),
                     scatter_lds(nx_max), s, e, i, n);
  return hipGetLastError();
}

hipError_t launch_sort(const SortArgs* a, int n, int num_cu, hipStream_t s) {
  if (n < 1 || n > 2 || a[0].nblocks > kMaxSortBlocks || (n == 2 && a[1].nblocks != a[0].nblocks))
    return hipErrorInvalidValue;
  SortPair p{{a[0], a[n - 1]}};
  const SortShape c = sort_chunks(&p.a[0], &p.a[1], 1, a->nx, num_cu);
  const dim3 g((unsigned)c.blocks, n);
  hipLaunchKernelGGL(k_sort_count, g, dim3(kSortThreads), (size_t)(a->nx - 1) * 4, s, p);
  hipLaunchKernelGGL(k_sort_scan, dim3(scan_blocks(a->nx, c.lanes), n), dim3(kSortThreads), 0, s, p,
                     c.lanes);
  hipLaunchKernelGGL(k_sort_scatter, g, dim3(kScatThreads), scatter_lds(a->nx), s, p);
  return hipGetLastError();
}

// The pool in slot order without moving the slots: entry i of the new pool
// is slot i's (v_y, v_z), and slot i's index becomes i.
__global__ __launch_bounds__(kSortThreads) void k_repack(SortArgs a) {
  const int64_t n = min(*a.count, a.cap);
  if (blockIdx.x == 0 && threadIdx.x == 0) *a.pool_n = n;
  for (int64_t i = (int64_t)blockIdx.x * kSortThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kSortThreads) {
    const uint32_t id = a.sid[i];
    a.dpv[i] = a.spv[id];
    a.did[i] = (uint32_t)i;
  }
}

hipError_t launch_repack(const SortArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_repack, dim3(1024), dim3(kSortThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace pic
