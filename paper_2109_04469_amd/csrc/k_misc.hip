// Small kernels: a species replaced (pic_set_state, pic_load_profile), the
// reading calls' reports, and the device self-checks of the generator and of
// FP64 sqrt.
#include "pic_internal.h"

namespace pic {

// A species replaced by n particles, in two launches. k_install_begin: the
// count and pool fill level, the cleared deposit, counters and error word, and
// (when the step parity changes) the other species' count on the new parity.
__global__ __launch_bounds__(256) void k_install_begin(InstallArgs a) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < a.nx) a.dep[i] = 0;
  if (i < kCounterSlots * NCOUNTERS) (&a.ctl->counters[0][0])[i] = 0ull;
  if (i == 0) {
    a.ctl->err = 0u;
    int64_t* own = a.species == 0 ? a.ctl->n_e : a.ctl->n_i;
    int64_t* other = a.species == 0 ? a.ctl->n_i : a.ctl->n_e;
    own[a.par] = a.n;
    *a.pool_n = a.n;
    if (a.old_par != a.par) other[a.par] = other[a.old_par];
  }
}

// A workgroup's share of the particles: pool entry and index per slot, and
// the deposit, summed in LDS and flushed once (2 n device-scope atomics on
// a few hundred addresses took 54 us for 30 thousand particles and 1.95 ms
// for 4 million).
template <bool HIST>
__device__ __forceinline__ void install_deposit(const InstallArgs& a, unsigned long long* sH,
                                                double x) {
  int j;
  double f;
  int64_t w1;
  cell_of(x, a.inv_dx, a.nx, j, f, w1);
  unsigned long long* d = HIST ? sH : reinterpret_cast<unsigned long long*>(a.dep);
  atomicAdd(&d[j], (unsigned long long)(kOne32 - w1));
  atomicAdd(&d[j + 1], (unsigned long long)w1);
}

__device__ __forceinline__ void install_flush(const InstallArgs& a, const unsigned long long* sH) {
  __syncthreads();
  for (int j = threadIdx.x; j < a.nx; j += 256)
    if (sH[j]) atomicAdd(reinterpret_cast<unsigned long long*>(&a.dep[j]), sH[j]);
}

__global__ __launch_bounds__(256) void k_install(InstallArgs a) {
  extern __shared__ unsigned long long sH[];
  for (int j = threadIdx.x; j < a.nx; j += 256) sH[j] = 0ull;
  __syncthreads();
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < a.n;
       i += (int64_t)gridDim.x * 256) {
    const double x = a.sx[i];
    if (a.sx != a.x) {
      a.x[i] = x;
      a.vx[i] = a.svx[i];
    }
    a.id[i] = (uint32_t)i;
    a.pv[i] = make_double2(a.svy[i], a.svz[i]);
    install_deposit<true>(a, sH, x);
  }
  install_flush(a, sH);
}

// workgroups of a launch over n particles: enough to fill the chip, few
// enough that the flushes of their histograms stay small
static unsigned install_grid(int64_t n) {
  const int64_t g = (n + 1023) / 1024;
  return (unsigned)(g < 1 ? 1 : g > 1024 ? 1024 : g);
}

hipError_t launch_install_begin(const InstallArgs& a, hipStream_t s) {
  const int n = a.nx > kCounterSlots * NCOUNTERS ? a.nx : kCounterSlots * NCOUNTERS;
  hipLaunchKernelGGL(k_install_begin, dim3((n + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_install(const InstallArgs& a, hipStream_t s) {
  if (a.n > 0)
    hipLaunchKernelGGL(k_install, dim3(install_grid(a.n)), dim3(256), (size_t)a.nx * 8, s, a);
  return hipGetLastError();
}

// Particles loaded from a density and a temperature profile given at npts
// equally spaced points on [0, L], both linear in between. Slot i takes the
// position whose cumulative density is u * (total) for its position uniform
// u (inverse of the piecewise-quadratic cumulative function, solved in
// closed form within the interval), and normal velocity components of
// variance e T(x) / m. Every workgroup builds the cumulative masses of the
// intervals in LDS in one fixed order: the masses in parallel, their sum by
// one thread, whose additions are a serial chain by definition (eight masses
// read ahead of them). HIST: the deposit is summed in LDS as in k_install,
// behind the cumulative masses.
template <bool HIST>
__global__ __launch_bounds__(256) void k_load_profile(LoadArgs a, InstallArgs p) {
  extern __shared__ double sC[];  // sC[k]: mass of the intervals below point k
  unsigned long long* sH = reinterpret_cast<unsigned long long*>(sC + a.npts);
  const int np = a.npts;
  if (HIST)
    for (int j = threadIdx.x; j < p.nx; j += 256) sH[j] = 0ull;
  for (int k = threadIdx.x; k + 1 < np; k += 256)
    sC[k + 1] = (fmax(a.dens[k], 0.0) + fmax(a.dens[k + 1], 0.0)) * a.hh;
  __syncthreads();
  if (threadIdx.x == 0) {
    double c = 0.0;
    sC[0] = 0.0;
    int k = 1;
    for (; k + 8 <= np; k += 8) {
      double m[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) m[q] = sC[k + q];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        c = c + m[q];
        sC[k + q] = c;
      }
    }
    for (; k < np; ++k) {
      c = c + sC[k];
      sC[k] = c;
    }
  }
  __syncthreads();
  const double total = sC[np - 1];
  const double h = a.h;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < p.n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint4 r0 = philox(make_uint4(kLoadStep, (uint32_t)i, 16u * a.species, 0u), a.seed, a.run);
    const double r = u01(r0.x) * total;
    // the last interval whose cumulative mass starts at or below r
    int lo = 0, hi = np - 2;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (sC[mid] <= r) lo = mid;
      else hi = mid - 1;
    }
    const double rp = r - sC[lo];
    const double da = fmax(a.dens[lo], 0.0), db = fmax(a.dens[lo + 1], 0.0);
    const double den = da + sqrt(fmax(da * da + 2.0 * (db - da) * rp / h, 0.0));
    double t = den > 0.0 ? 2.0 * rp / den : 0.0;
    t = fmin(fmax(t, 0.0), h);
    const double x = fmin((double)lo * h + t, a.L);
    const double ta = a.temp[lo], tb = a.temp[lo + 1];
    const double T = fmax(ta + (tb - ta) * (t / h), 0.0);
    const double sig = sqrt(T * a.vfac);
    const uint4 r1 = philox(make_uint4(kLoadStep, (uint32_t)i, 16u * a.species + 1u, 0u), a.seed,
                            a.run);
    double n1, n2, n3, n4;
    box_muller(u01(r1.x), u01(r1.y), n1, n2);
    box_muller(u01(r1.z), u01(r1.w), n3, n4);
    p.x[i] = x;
    p.vx[i] = sig * n1;
    p.pv[i] = make_double2(sig * n2, sig * n3);
    p.id[i] = (uint32_t)i;
    install_deposit<HIST>(p, sH, x);
  }
  if (HIST) install_flush(p, sH);
}

hipError_t launch_load_profile(const LoadArgs& a, const InstallArgs& p, hipStream_t s) {
  if (a.npts < 2 || a.npts > kMaxLoadPoints) return hipErrorInvalidValue;
  if (p.n < 1) return hipSuccess;
  // both tables in LDS up to 64 KB, what a workgroup may have beside another
  // one; longer profiles on larger grids deposit straight to memory
  const size_t both = ((size_t)a.npts + (size_t)p.nx) * 8;
  if (both <= 65536)
    hipLaunchKernelGGL(k_load_profile<true>, dim3(install_grid(p.n)), dim3(256), both, s, a, p);
  else
    hipLaunchKernelGGL(k_load_profile<false>, dim3(install_grid(p.n)), dim3(256),
                       (size_t)a.npts * 8, s, a, p);
  return hipGetLastError();
}

__global__ void k_selftest_philox(const uint32_t* ctr, uint32_t k0, uint32_t k1, uint32_t* out,
                                  int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint4 r = philox(make_uint4(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3]),
                         k0, k1);
  out[4 * i] = r.x;
  out[4 * i + 1] = r.y;
  out[4 * i + 2] = r.z;
  out[4 * i + 3] = r.w;
}

__global__ void k_selftest_sqrt(const double* in, double* out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = sqrt(in[i]);
}

// The words every report starts with, by the first threads of a workgroup.
__device__ __forceinline__ void report_words(const ReportArgs& a) {
  const DevCtl* c = a.ctl;
  const int t = threadIdx.x;
  if (t == 0) a.out[R_ERR] = c->err;
  if (t == 1) a.out[R_NE] = (uint64_t)c->n_e[a.par];
  if (t == 2) a.out[R_NI] = (uint64_t)c->n_i[a.par];
  if (t == 3) a.out[R_MSTEPS] = (uint64_t)c->msteps;
  if (t == 4 || t == 5) a.out[R_NCODES_E + t - 4] = (uint64_t)c->ncodes[t - 4];
  if (t >= 8 && t < 12) a.out[R_HITS + t - 8] = (&c->wall_hits[0][0])[t - 8];
  if (t >= 12 && t < 16) a.out[R_ABSORBED + t - 12] = (&c->wall_absorbed[0][0])[t - 12];
  if (t >= 16 && t < 20)
    a.out[R_ESUM + t - 16] = (uint64_t)__double_as_longlong((&c->wall_esum[0][0])[t - 16]);
  if (t == 20) a.out[R_IONIZ] = c->ioniz_meas;
}

// A reading call costs one launch and one wait, whatever it reads (copies
// into pageable memory cost about 20 us each with their wait: a state, its
// count and the error word were six of them).
__global__ __launch_bounds__(256) void k_report(ReportArgs a) {
  if (blockIdx.x == 0) {
    report_words(a);
    if (a.counters) {
      __shared__ unsigned long long sum[NCOUNTERS];
      if (threadIdx.x < NCOUNTERS) sum[threadIdx.x] = 0ull;
      __syncthreads();
      unsigned long long v = 0ull;
      for (int k = threadIdx.x / NCOUNTERS; k < kCounterSlots; k += 256 / NCOUNTERS)
        v += a.ctl->counters[k][threadIdx.x % NCOUNTERS];
      atomicAdd(&sum[threadIdx.x % NCOUNTERS], v);
      __syncthreads();
      if (threadIdx.x < NCOUNTERS) a.out[R_COUNTERS + threadIdx.x] = sum[threadIdx.x];
    }
    return;
  }
  uint64_t* out = a.out + R_ARRAYS;
#pragma unroll
  for (int k = 0; k < kReportArrays; ++k) {
    const uint64_t* src = static_cast<const uint64_t*>(a.src[k]);
    for (int i = (blockIdx.x - 1) * 256 + threadIdx.x; i < a.n[k]; i += (gridDim.x - 1) * 256)
      out[i] = src[i];
    out += a.n[k];
  }
}

hipError_t launch_report(const ReportArgs& a, hipStream_t s) {
  int most = 0;
  for (int k = 0; k < kReportArrays; ++k) most = a.n[k] > most ? a.n[k] : most;
  hipLaunchKernelGGL(k_report, dim3(1 + (most + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

__global__ __launch_bounds__(64) void k_counts(const DevCtl* c, int par, int64_t* out) {
  if (threadIdx.x == 0) out[0] = c->n_e[par];
  if (threadIdx.x == 1) out[1] = c->n_i[par];
}

__global__ __launch_bounds__(kMaxBatch) void k_batch_counts(const BatchCount* c, int n,
                                                            int64_t* out) {
  const int d = threadIdx.x;
  if (d >= n) return;
  out[2 * d] = c[d].ctl->n_e[c[d].par];
  out[2 * d + 1] = c[d].ctl->n_i[c[d].par];
}

hipError_t launch_batch_counts(const BatchCount* c, int n, int64_t* out, hipStream_t s) {
  if (n < 1 || n > kMaxBatch) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_batch_counts, dim3(1), dim3(kMaxBatch), 0, s, c, n, out);
  return hipGetLastError();
}

hipError_t launch_counts(const DevCtl* ctl, int par, int64_t* out, hipStream_t s) {
  hipLaunchKernelGGL(k_counts, dim3(1), dim3(64), 0, s, ctl, par, out);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_export(ExportArgs e, ReportArgs a) {
  if (blockIdx.x == 0) report_words(a);
  const DevCtl* c = a.ctl;
  const int64_t n = e.species == 0 ? c->n_e[a.par] : c->n_i[a.par];
  if (c->err || n > e.cap) return;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const double2 v = e.pool[e.id[i]];
    e.out[0][i] = e.x[i];
    e.out[1][i] = e.vx[i];
    e.out[2][i] = v.x;
    e.out[3][i] = v.y;
  }
}

hipError_t launch_export(const ExportArgs& e, const ReportArgs& a, hipStream_t s) {
  int64_t g = (e.cap + 255) / 256;
  if (g > 2048) g = 2048;
  if (g < 1) g = 1;
  hipLaunchKernelGGL(k_export, dim3((unsigned)g), dim3(256), 0, s, e, a);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_clear(ClearArgs a) {
#pragma unroll
  for (int k = 0; k < 10; ++k)
    for (int i = blockIdx.x * 256 + threadIdx.x; i < a.n[k]; i += gridDim.x * 256) a.p[k][i] = 0ull;
}

hipError_t launch_clear(const ClearArgs& a, hipStream_t s) {
  int most = 1;
  for (int n : a.n) most = n > most ? n : most;
  hipLaunchKernelGGL(k_clear, dim3((most + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_clear2(int64_t* a, int64_t* b, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) a[i] = b[i] = 0;
}

hipError_t launch_clear2(int64_t* a, int64_t* b, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_clear2, dim3((n + 255) / 256), dim3(256), 0, s, a, b, n);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_gather(const uint32_t* id, const double2* pool,
                                                double* out_y, double* out_z, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double2 v = pool[id[i]];
    out_y[i] = v.x;
    out_z[i] = v.y;
  }
}

hipError_t launch_gather(const uint32_t* id, const double2* pool, double* out_y, double* out_z,
                         int64_t n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_gather, dim3(1024), dim3(256), 0, s, id, pool, out_y, out_z, n);
  return hipGetLastError();
}

// Plain streaming copy, 16 bytes per lane per iteration: the reference
// kernel for achievable HBM bandwidth and for scaling traffic counters.
__global__ __launch_bounds__(256) void k_selftest_copy(const double2* __restrict__ in,
                                                        double2* __restrict__ out, int64_t n2) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n2; i += stride)
    out[i] = in[i];
}

hipError_t launch_selftest_copy(const double* in, double* out, int64_t n, hipStream_t s) {
  const int64_t n2 = n / 2;
  int64_t g = (n2 + 255) / 256;
  if (g > 65536) g = 65536;
  if (g > 0)
    hipLaunchKernelGGL(k_selftest_copy, dim3((unsigned)g), dim3(256), 0, s,
                       reinterpret_cast<const double2*>(in), reinterpret_cast<double2*>(out), n2);
  return hipGetLastError();
}

hipError_t launch_selftest_philox(const uint32_t* ctr, uint32_t k0, uint32_t k1, uint32_t* out,
                                  int64_t n, hipStream_t s) {
  const int64_t g = (n + 255) / 256;
  if (g > 0) hipLaunchKernelGGL(k_selftest_philox, dim3((unsigned)g), dim3(256), 0, s, ctr, k0, k1, out, n);
  return hipGetLastError();
}

hipError_t launch_selftest_sqrt(const double* in, double* out, int64_t n, hipStream_t s) {
  const int64_t g = (n + 255) / 256;
  if (g > 0) hipLaunchKernelGGL(k_selftest_sqrt, dim3((unsigned)g), dim3(256), 0, s, in, out, n);
  return hipGetLastError();
}

}  // namespace pic
