// One-kernel step: the emit of step n and the decisions of step n + 1 for
// both species in one launch (arXiv:2109.04469, Sec. 2 steps 1-6).
//
// The per-pass kernels (k_particle.hip) take six launches for a step on
// which both species move: electron decide, emit and queued slots, ion
// decide and emit, and the tail with the next field. On anything but the
// largest discharges each of them is a chain of latencies (start-up, counts,
// field staging, a tile's loads, the collision chain) that leaves most of
// the chip idle. Here everything of a step that only depends on the previous
// launch runs in one:
//   * the field of step n + 1 is solved by every workgroup for itself from
//     the finished deposits (grids up to kSelfMaxNx nodes; an exact integer
//     prefix form, so all workgroups get the same bits), or staged from the
//     field kernel's result;
//   * both species' tiles are laid end to end over the workgroups. A tile's
//     slots are compacted in slot order to their output slots, found from the
//     tile totals that the previous launch left, and every output is pushed
//     and decided for step n + 1 at once;
//   * slots that need draws (collision kinematics, emission) and outputs
//     that leave the gap or are electron collision candidates go to a queue
//     in LDS, one per wave: a wave takes 64 of a kind at a time, so that no
//     lane idles through these chains of dependent loads and no other wave
//     waits for them; what is left after the last tile is shared by the
//     workgroup, queued slots from the first thread up, deferred outputs
//     from the last thread down;
//   * births are written straight to their slots in the other species'
//     output (after its survivors, whose number is the sum of its tile
//     totals) and decided there.
// Nothing a launch reads is written by it: counts and pool fill levels are
// double-buffered, tile totals and deposits triple-buffered (read, added
// into, zeroed for the launch after). Every decision uses the same
// arithmetic and draws as the per-pass kernels, so results are the same
// bits whichever path takes a step.
#include <climits>

#include "field_block.h"
#include "particle_dev.h"
#include "pic_internal.h"

namespace pic {

constexpr int kStepWaves = kBlock / kWave;
// Waves per SIMD the register budget must allow: at the compiler's own choice
// (176 registers, two waves) the 64-discharge sweep took 68.2 ms per 40
// steps, with three (168 registers) 57.6 ms, with four (128, spilled) 71.4.
constexpr int kStepMinWaves = 3;
// The method variants' collision (pow, tan, atan) needs more registers than
// the rest of the step. Inlined, the 2048-slot instances held 256 and more: one
// wave per SIMD. There it is a call of its own, made by the few slots that
// collide, and the instances keep three waves. us per step, inlined / inlined
// and held to two waves / to three (77 to 99 spilled) / called: 2 million of
// each species on 512 cells 69 / 48 / 65 / 48, measuring 98 / 69 / 91 / 68; the
// 64-discharge sweep with one discharge of them so 1026 / 663 / 694 / 657,
// measuring 1463 / 875 / 862 / 765. The 512-slot instances, two waves with it
// inlined, keep it so: up to 50 thousand of each species the call costs more
// than the waves give (16.4 against 17.1).
constexpr bool step_calls_variant(int ppt) { return ppt == kStepPpt[0]; }
constexpr int step_min_waves(int ppt, bool var) {
  return var && !step_calls_variant(ppt) ? 1 : kStepMinWaves;
}
constexpr int kStepOrd = 16;  // a queue entry names its tile in four bits
constexpr int kStepTally = 64;  // output tiles whose totals a workgroup sums in LDS

// The argument block, read through the scalar cache. Its pointers are to
// global memory, which gptr tells the compiler (no flat accesses), and
// fresh() ends the life of values read before it: the block is far larger
// than the scalar register file. Between those points the compiler still
// spills 250 to 400 scalars per instance to lanes of vector registers, the
// schedule's flags and the addresses of two species among them.
typedef const __attribute__((address_space(4))) StepArgs CArgs;
typedef const __attribute__((address_space(4))) StepSpecies CSpecies;

template <typename T>
__device__ __forceinline__ T* gptr(T* p) {
  return (T*)(__attribute__((address_space(1))) T*)p;
}

__device__ __forceinline__ CArgs& fresh(CArgs& a) {
  CArgs* p = &a;
  asm volatile("" : "+s"(p));
  return *p;
}

template <int PPT>
struct StepTile {
  static constexpr int kSlots = kBlock * PPT;
  static constexpr int kPairs = PPT / 2;
  static constexpr int kBlocks = 2 * kSlots / 4 + 4;  // draw blocks of a tile's outputs
  // a wave's queue: less than a wave's worth of each kind carried over, and
  // every slot of its quarter of a tile
  static constexpr int kQueue = kSlots / kStepWaves + 2 * kWave;
  static_assert(PPT % 2 == 0 && kSlots <= 2048, "pairs of slots, 9-bit slots in a queue entry");
};

// Totals of the emitted step and where its births go. In LDS: only slots with
// a birth need them.
struct StepTotals {
  int64_t ion0;     // slot of the first ionization ion
  int64_t se0;      // slot of the first secondary electron
  int64_t pe, pi;   // first pool entries of the ionizations
  int64_t pse;      // first pool entry of the secondary electrons
};

template <int PPT>
struct StepShared {
  using T = StepTile<PPT>;
  uint64_t q[kStepWaves][T::kQueue];  // queued slots from the front, deferred outputs from the back
  unsigned long long cnt[NCOUNTERS];
  i128p w128[kStepWaves];
  int64_t w64[kStepWaves];
  uint32_t red[8][kStepWaves];
  uint32_t wtot[2][T::kPairs][kStepWaves];  // two copies, used by alternate tiles
  uint8_t cand[2][T::kBlocks];  // candidacy bits of four output slots each
  uint32_t pref[kStepWaves][kStepOrd][3];  // outputs and births before a queue entry's tile, the tile
  uint32_t tally[kStepTally];
  uint32_t left[2][kStepWaves];  // entries left in each wave's queue
  StepTotals tot;
};

// The workgroup's LDS: the fixed part, then the grids of ld nodes each.
extern __shared__ __align__(16) unsigned char step_smem[];

template <int PPT>
struct StepLds {
  int ld;
  __device__ __forceinline__ StepShared<PPT>& s() const {
    return *reinterpret_cast<StepShared<PPT>*>(step_smem);
  }
  // field of the decided step, deposit, energy averages and EEPF (measuring)
  __device__ __forceinline__ double* E() const {
    return reinterpret_cast<double*>(step_smem + sizeof(StepShared<PPT>));
  }
  __device__ __forceinline__ unsigned long long* H() const {
    return reinterpret_cast<unsigned long long*>(E() + ld);
  }
  __device__ __forceinline__ double* EW() const { return E() + 2 * ld; }
  __device__ __forceinline__ uint32_t* EEPF() const {
    return reinterpret_cast<uint32_t*>(E() + 3 * ld);
  }
};

// A queue entry: the slot within the wave's share of its tile (9 bits), the
// output offset within the tile (13), the tile's place in StepShared::pref
// (4), a deferred output's candidacy (1), a queued slot's process (3), and in
// the upper half the pool index, so that the velocity pool is read together
// with the particle; a slot with a birth has the birth's rank there instead.
constexpr uint32_t kProcIon = 1u;   // Ar+ candidate (electrons: the process, 2 to 4)
constexpr uint32_t kProcEmit = 7u;  // Ar+ impact that emits an electron

__device__ __forceinline__ uint64_t step_entry(uint32_t local, uint32_t off, uint32_t ord,
                                               bool cand, uint32_t proc, uint32_t hi) {
  return (uint64_t)(local | (off << 9) | (ord << 22) | (cand ? 1u << 26 : 0u) | (proc << 27)) |
         ((uint64_t)hi << 32);
}

// ---------------------------------------------------------------------------
// The exact field solve (field_block.h) by one workgroup of kBlock threads:
// the same integers and the same roundings per node, E into LDS. lead: also
// the stores of rho, phi, E and the density averages.
template <int kMaxNodes>
__device__ __forceinline__ void step_field(CArgs& a, double* sE, i128p* s128, int64_t* s64,
                                           bool lead) {
  constexpr int kOwn = (kMaxNodes - 1 + kBlock - 1) / kBlock + 1;  // nodes of a thread
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = tid / kWave;
  const int nx = a.nx;
  const int m = nx - 1;
  const int per = (m + kBlock - 1) / kBlock;
  const int j0 = tid * per;
  const int j1 = tid == kBlock - 1 ? nx : min(j0 + per, nx);
  int64_t de[kOwn], c[kOwn], loc[kOwn];
  {
    int64_t di[kOwn];
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      const int j = j0 + q;
      de[q] = j < j1 ? gptr(a.sp[0].dep_in)[j] : 0;
      di[q] = j < j1 ? gptr(a.sp[1].dep_in)[j] : 0;
    }
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      c[q] = di[q] - de[q];
      const int j = j0 + q;
      if (lead && j < j1) {
        const bool wall = (j == 0) || (j == nx - 1);
        double r = (double)c[q] * a.qfac32;
        if (wall) r = 2.0 * r;
        gptr(a.rho)[j] = r;
        // ions that are not pushed keep their deposit
        if (!a.sp[1].decide) atomicAdd(&gptr(a.sp[1].dep_out)[j], (unsigned long long)di[q]);
        if (a.measuring) {
          double ne = (double)de[q] * a.nfac32;
          double ni = (double)di[q] * a.nfac32;
          if (wall) {
            ne = 2.0 * ne;
            ni = 2.0 * ni;
          }
          // one addition per node and launch: nothing to wait for (50 steps of
          // 400 thousand particles 1.91 -> 1.88 ms against reading and writing
          // back, which held up the workgroup that leads a discharge)
          atomicAdd(&gptr(a.acc_ne)[j], ne);
          atomicAdd(&gptr(a.acc_ni)[j], ni);
          atomicAdd(&gptr(a.acc_w)[j], (double)de[q] * kInvTwo32);
        }
      }
    }
  }
  int64_t s = 0;
#pragma unroll
  for (int q = 0; q < kOwn; ++q) {
    const int k = j0 + q;
    if (k < j1 && k < m && k >= 1) s += c[q];
    loc[q] = s;
  }
  const int64_t inc = wave_incl_scan64(s);
  if (lane == kWave - 1) s64[wave] = inc;
  __syncthreads();
  int64_t qb = inc - s;
#pragma unroll
  for (int w = 0; w < kStepWaves; ++w) qb += w < wave ? s64[w] : 0;
  i128p rsum = from64(0);
#pragma unroll
  for (int q = 0; q < kOwn; ++q)
    if (j0 + q < j1 && j0 + q < m) rsum = add128(rsum, from64(qb + loc[q]));
  const i128p rinc = wave_incl_scan128(rsum);
  if (lane == kWave - 1) s128[wave] = rinc;
  __syncthreads();
  i128p rb = from64(0), rtot = from64(0);
#pragma unroll
  for (int w = 0; w < kStepWaves; ++w) {
    if (w < wave) rb = add128(rb, s128[w]);
    rtot = add128(rtot, s128[w]);
  }
  const double K = a.kpois;
  const double dx = a.dx;
  const double V = a.V;
  const double D0 = (K * to_double(rtot) - V) / (double)(nx - 1);
  int64_t qprev = qb;
#pragma unroll
  for (int q = 0; q < kOwn; ++q) {
    const int j = j0 + q;
    if (j >= j1) continue;
    const int64_t qj = qb + loc[q];
    double e;
    if (j == 0 || j == nx - 1) {
      const double r = 2.0 * ((double)c[q] * a.qfac32);
      if (j == 0) {
        e = -D0 / dx - r * dx / (2.0 * kEps0);
      } else {
        const double Dlast = D0 - K * (double)qprev;
        e = -Dlast / dx + r * dx / (2.0 * kEps0);
      }
    } else {
      e = (K * (double)(qprev + qj) - 2.0 * D0) / (2.0 * dx);
    }
    sE[j] = e;
    qprev = qj;
  }
  if (lead) {
    // phi needs R at this thread's nodes: the exclusive scan of rsum
    i128p neg;
    neg.lo = ~rsum.lo + 1;
    neg.hi = ~rsum.hi + (neg.lo == 0 ? 1 : 0);
    i128p r = add128(add128(rb, rinc), neg);
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      const int j = j0 + q;
      if (j >= j1) continue;
      if (j < m) {
        gptr(a.phi)[j] = V + (double)j * D0 - K * to_double(r);
        r = add128(r, from64(qb + loc[q]));
      } else {
        gptr(a.phi)[j] = 0.0;
      }
      gptr(a.E)[j] = sE[j];
      if (!isfinite(sE[j])) latch_error(gptr(a.ctl), kErrUnstable);
    }
  }
}

// ---------------------------------------------------------------------------
// decisions of single outputs

// A particle of species SP reaching electrode `wall` with the pushed
// velocity: arrival count, absorption, impact energy and its bin (Sec. 3.3).
template <int SP>
__device__ __forceinline__ void step_arrival(CArgs& a, double vx, double vy, double vz,
                                             int wall, bool absorbed) {
  CSpecies& s = a.sp[SP];
  const double eps = s.ek_s * (vx * vx + vy * vy + vz * vz);
  DevCtl* ctl = gptr(a.ctl);
  atomicAdd(&ctl->wall_hits[SP][wall], 1ull);
  if (absorbed) atomicAdd(&ctl->wall_absorbed[SP][wall], 1ull);
  atomicAdd(&ctl->wall_esum[SP][wall], eps);
  const int64_t bin = (int64_t)(eps * s.fedf_inv_de);
  if (bin >= 0 && bin < a.nbins) atomicAdd(&gptr(s.fedf)[(int64_t)wall * a.nbins + bin], 1ull);
}

// Left the gap, or not finite: a velocity that is not finite leaves a
// position that is not, either.
__device__ __forceinline__ bool step_outside(CArgs& a, double x) {
  return !(x >= 0.0 && x <= a.L);
}

// The wall model and the collision decision of one pushed output that left
// the gap or is a collision candidate. vy, vz: used for candidate electrons
// and arrivals. The code, the outputs and the births come back in c, o, b.
template <int SP, int PPT>
__device__ __forceinline__ void step_need(CArgs& a, StepLds<PPT> S, int64_t slot,
                                          bool cand, double& x, double& vx, double vy, double vz,
                                          uint32_t& c, uint32_t& o, uint32_t& b) {
  const double L = a.L;
  bool alive = true;
  uint32_t mul = 1;
  if (!isfinite(x) || !isfinite(vx)) {
    latch_error(gptr(a.ctl), kErrUnstable);
    alive = false;
    c |= 1u;
  } else if (x < 0.0 || x > L) {
    const int wall = x < 0.0 ? 0 : 1;
    const double vx_hit = vx;
    const double ub = u01(draw(a.dstep, (uint32_t)slot, SP, 0, a.seed, a.run).x);
    if (SP == 0) {
      if (ub < a.sp[0].p_wall) {
        x = (x < 0.0) ? -x : (L + L) - x;
        vx = -vx;
        if (x < 0.0 || x > L) {
          alive = false;
          c |= 4u;
          atomicAdd(&S.s().cnt[C_REFLECT_LOST], 1ull);
        } else {
          c |= 2u;
          atomicAdd(&S.s().cnt[C_E_REFLECTED], 1ull);
        }
      } else {
        alive = false;
        c |= 1u;
        atomicAdd(&S.s().cnt[C_E_ABSORBED], 1ull);
      }
    } else {
      alive = false;
      atomicAdd(&S.s().cnt[C_I_ABSORBED], 1ull);
      if (ub < a.sp[1].p_wall) {
        // a secondary electron leaves the wall the ion hit
        c |= 3u;
        b = 1;
        atomicAdd(&S.s().cnt[C_SE_EMITTED], 1ull);
        deposit_global(gptr(a.sp[0].dep_out), x < 0.0 ? 0.0 : L, a.inv_dx, a.nx);
      } else {
        c |= 1u;
      }
    }
    if (a.measuring) step_arrival<SP>(a, vx_hit, vy, vz, wall, !alive);
  }
  if (alive && cand) {
    if (SP == 0) {
      // the process at this speed decides whether a second electron and an
      // ion are born
      atomicAdd(&S.s().cnt[C_E_CAND], 1ull);
      CSpecies& s = a.sp[0];
      const double g2 = sqrt(vx * vx + vy * vy + vz * vz);
      const double tv = g2 * s.inv_dv;
      // the three cumulative frequencies read together: one round trip
      const double n0 = cum_nu<3>(gptr(s.cum), a.ntab, 0, tv);
      const double n1 = cum_nu<3>(gptr(s.cum), a.ntab, 1, tv);
      const double n2 = cum_nu<3>(gptr(s.cum), a.ntab, 2, tv);
      const double r = u01(draw(a.dstep, (uint32_t)slot, 0, 0, a.seed, a.run).z) * s.numax;
      if (!(tv < (double)(a.ntab - 1))) atomicAdd(&S.s().cnt[C_BEYOND_TABLE], 1ull);
      uint32_t proc = 1;
      if (r < n0) {
        proc = 2;
        atomicAdd(&S.s().cnt[C_E_ELASTIC], 1ull);
      } else if (r < n1) {
        proc = 3;
        atomicAdd(&S.s().cnt[C_E_EXC], 1ull);
      } else if (r < n2) {
        proc = 4;
        b = 1;
        mul = 2;
        atomicAdd(&S.s().cnt[C_E_ION], 1ull);
        if (a.measuring) atomicAdd(&gptr(a.ctl)->ioniz_meas, 1ull);
        deposit_global(gptr(a.sp[1].dep_out), x, a.inv_dx, a.nx);
      }
      c |= proc << 3;
    } else {
      atomicAdd(&S.s().cnt[C_I_CAND], 1ull);
      c |= kIonPending;
    }
  }
  o = alive ? mul : 0u;
}

// An electron's share of the energy averages at the start of the decided
// step: CIC-weighted energy at x's cell (j, w1), and its EEPF bin. run: the
// caller's run of shares at the nodes (cell, cell + 1), added when the cell
// changes (sorted particles: the two of a pair nearly always share a cell).
struct EnergyRun {
  int cell;
  double e0, e1;
};

template <int PPT>
__device__ __forceinline__ void step_energy_flush(StepLds<PPT> S, const EnergyRun& run) {
  if (run.cell >= 0) {
    atomicAdd(&S.EW()[run.cell], run.e0);
    atomicAdd(&S.EW()[run.cell + 1], run.e1);
  }
}

template <int PPT>
__device__ __forceinline__ void step_energy(CArgs& a, StepLds<PPT> S, double x, int j, int64_t w1,
                                            double eps, EnergyRun& run) {
  const double s0 = ((double)(kOne32 - w1) * kInvTwo32) * eps;
  const double s1 = ((double)w1 * kInvTwo32) * eps;
  if (j == run.cell) {
    run.e0 += s0;
    run.e1 += s1;
  } else {
    step_energy_flush(S, run);
    run = EnergyRun{j, s0, s1};
  }
  if (fabs(x - a.half) <= a.eepf_hw) {
    const int64_t bin = (int64_t)(eps * a.inv_de);
    if (bin >= 0 && bin < a.nbins) atomicAdd(&S.EEPF()[bin], 1u);
  }
}

// Adds one output slot's outcome to the tile totals of the decided step.
// OWN: the workgroup's own run of outputs, summed in LDS from tile ta0 on,
// where every output slot has been counted as one plain output beforehand
// (step_tiles): o is what comes on top, modulo 2^32.
template <int SP, int PPT, bool OWN>
__device__ __forceinline__ void step_tally(CArgs& a, StepLds<PPT> S, int64_t dest,
                                           uint32_t ta0, uint32_t o, uint32_t b) {
  const uint32_t w = o + (b << 16);
  if (!w) return;
  const uint32_t tile = (uint32_t)((uint64_t)dest / StepTile<PPT>::kSlots);
  if (OWN && tile - ta0 < kStepTally)
    atomicAdd(&S.s().tally[tile - ta0], w);
  else
    atomicAdd(&gptr(a.sp[SP].tout)[tile], w);
}

// An output of the emitted step at slot dest (state after that step, pool
// entry written) taken through the decided step: push, candidacy, wall and
// collision decisions, code, tile totals, deposit and the pushed state.
// OWN: dest belongs to this workgroup's run (deposit and totals in LDS).
template <int SP, int PPT, bool MEASURE, bool OWN>
__device__ __forceinline__ void step_decide_one(CArgs& a, StepLds<PPT> S, int64_t dest,
                                                uint32_t ta0, double x, double vx, double vy,
                                                double vz, uint32_t id) {
  CSpecies& s = a.sp[SP];
  if (dest >= s.cap) return;
  if (!s.decide) {
    gptr(s.xout)[dest] = x;
    gptr(s.vxout)[dest] = vx;
    gptr(s.idout)[dest] = id;
    return;
  }
  int j;
  double f;
  int64_t w1;
  cell_of(x, a.inv_dx, a.nx, j, f, w1);
  if (MEASURE && SP == 0 && a.measuring) {
    EnergyRun run{-1, 0.0, 0.0};
    step_energy(a, S, x, j, w1, a.ek * (vx * vx + vy * vy + vz * vz), run);
    step_energy_flush(S, run);
  }
  push(S.E(), j, f, s.acc, s.dts, x, vx);
  bool cand = false;
  if (s.cand_thr) {
    const uint4 r = draw(a.dstep, (uint32_t)(dest >> 2), SP, 4, a.seed, a.run);
    const uint32_t k = (uint32_t)dest & 3u;
    const uint32_t w = k == 0u ? r.x : k == 1u ? r.y : k == 2u ? r.z : r.w;
    cand = (uint64_t)w < s.cand_thr;
  }
  uint32_t c = kCodePushed, o = 1u, b = 0u;
  if (cand || step_outside(a, x))
    step_need<SP, PPT>(a, S, dest, cand, x, vx, vy, vz, c, o, b);
  gptr(s.cout)[dest] = (uint8_t)c;
  step_tally<SP, PPT, OWN>(a, S, dest, ta0, OWN ? o - 1u : o, b);
  if (o) {
    cell_of(x, a.inv_dx, a.nx, j, f, w1);
    const unsigned long long q0 = (unsigned long long)o * (unsigned long long)(kOne32 - w1);
    const unsigned long long q1 = (unsigned long long)o * (unsigned long long)w1;
    if (OWN) {
      atomicAdd(&S.H()[j], q0);
      atomicAdd(&S.H()[j + 1], q1);
    } else {
      atomicAdd(&gptr(s.dep_out)[j], q0);
      atomicAdd(&gptr(s.dep_out)[j + 1], q1);
    }
  }
  gptr(s.xout)[dest] = x;
  gptr(s.vxout)[dest] = vx;
  gptr(s.idout)[dest] = id;
}

// The slot, output slot and birth rank base of entry e of wave qw's queue.
template <int PPT>
__device__ __forceinline__ void step_place(StepLds<PPT> S, uint64_t e, int qw, int64_t& slot,
                                           int64_t& dest, uint32_t& births) {
  const uint32_t lo = (uint32_t)e;
  const uint32_t local = lo & 0x1FFu;
  const uint32_t* pf = S.s().pref[qw][(lo >> 22) & 15u];
  slot = (int64_t)pf[2] * StepTile<PPT>::kSlots +
         (int64_t)((local >> 7) * (2 * kBlock) + (uint32_t)qw * (2 * kWave) + (local & 127u));
  dest = (int64_t)pf[0] + (int64_t)((lo >> 9) & 0x1FFFu);
  births = pf[1];
}

// A variant collision out of line: the velocities after it of the electron, a
// second electron and an ion (electron_collision).
struct VariantCollision {
  double v[3], cv[3], bv[3];
  bool child;
};
__device__ __attribute__((noinline)) VariantCollision variant_collision(CArgs* a, uint32_t slot,
                                                                        uint32_t proc, double vx,
                                                                        double vy, double vz) {
  VariantCollision r{{vx, vy, vz}, {0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}, false};
  r.child = electron_collision<true>(*a, a->mstep, slot, proc, r.v[0], r.v[1], r.v[2], r.cv, r.bv);
  return r;
}

// One queued slot of the emitted step: collision kinematics, ion process or
// emission, and its outputs and births.
template <int SP, int PPT, bool MEASURE, bool VAR>
__device__ __forceinline__ void step_queued(CArgs& a, StepLds<PPT> S, uint64_t e, int qw,
                                            uint32_t ta0) {
  CSpecies& s = a.sp[SP];
  int64_t slot, dest;
  uint32_t births;
  step_place(S, e, qw, slot, dest, births);
  const uint32_t proc = ((uint32_t)e >> 27) & 7u;
  const uint32_t hi = (uint32_t)(e >> 32);
  const int64_t r = (int64_t)births + (int64_t)hi;  // slots with a birth
  const double x = gptr(s.xin)[slot];
  double cv[3] = {0.0, 0.0, 0.0}, bv[3] = {0.0, 0.0, 0.0};
  if (SP == 1 && proc == kProcEmit) {
    // secondary electron from the wall the ion hit
    double bx;
    secondary_electron(a, a.mstep, (uint32_t)slot, x, bx, bv);
    CSpecies& o = a.sp[0];
    const int64_t bd = S.s().tot.se0 + r, bid = S.s().tot.pse + r;
    if (bd < o.cap && bid < o.pcap) {
      gptr(o.pv)[bid] = make_double2(bv[1], bv[2]);
      step_decide_one<0, PPT, MEASURE, false>(a, S, bd, 0u, bx, bv[0], bv[1], bv[2],
                                              (uint32_t)bid);
    }
    return;
  }
  double vx = gptr(s.vxin)[slot];
  uint32_t id = hi;
  if (SP == 0 && proc == 4u) id = gptr(s.idin)[slot];
  const double2 pv = gptr(s.pv)[id];
  double vy = pv.x, vz = pv.y;
  if (SP == 0) {
    bool child;
    if constexpr (VAR && step_calls_variant(PPT)) {
      const VariantCollision vc = variant_collision(&a, (uint32_t)slot, proc, vx, vy, vz);
      vx = vc.v[0];
      vy = vc.v[1];
      vz = vc.v[2];
      for (int k = 0; k < 3; ++k) {
        cv[k] = vc.cv[k];
        bv[k] = vc.bv[k];
      }
      child = vc.child;
    } else {
      child = electron_collision<VAR>(a, a.mstep, (uint32_t)slot, proc, vx, vy, vz, cv, bv);
    }
    gptr(s.pv)[id] = make_double2(vy, vz);
    int64_t d = dest;
    for (int k = 0;; ++k) {
      step_decide_one<0, PPT, MEASURE, true>(a, S, d, ta0, x, vx, vy, vz, id);
      if (k == 1 || !child) break;
      // the ionization electron follows its parent, with a fresh pool entry
      const int64_t cid = S.s().tot.pe + r;
      d = dest + 1;
      if (cid >= s.pcap || d >= s.cap) break;
      vx = cv[0];
      vy = cv[1];
      vz = cv[2];
      id = (uint32_t)cid;
      gptr(s.pv)[cid] = make_double2(vy, vz);
    }
    if (child) {
      CSpecies& o = a.sp[1];
      const int64_t bd = S.s().tot.ion0 + r, bid = S.s().tot.pi + r;
      if (bd < o.cap && bid < o.pcap) {
        gptr(o.pv)[bid] = make_double2(bv[1], bv[2]);
        step_decide_one<1, PPT, MEASURE, false>(a, S, bd, 0u, x, bv[0], bv[1], bv[2],
                                                (uint32_t)bid);
      }
    }
  } else {
    bool beyond;
    const uint32_t k = ion_collision(a, a.mstep, (uint32_t)slot, gptr(s.cum), s.numax, s.inv_dv,
                                     vx, vy, vz, beyond);
    if (beyond) atomicAdd(&S.s().cnt[C_BEYOND_TABLE], 1ull);
    if (k == 2u) atomicAdd(&S.s().cnt[C_I_ISO], 1ull);
    if (k == 3u) atomicAdd(&S.s().cnt[C_I_BACK], 1ull);
    gptr(s.cin)[slot] = (uint8_t)((uint32_t)kCodePushed | (k << 3));
    gptr(s.pv)[id] = make_double2(vy, vz);
    step_decide_one<1, PPT, MEASURE, true>(a, S, dest, ta0, x, vx, vy, vz, id);
  }
}

// An output that left the gap or is an electron candidate: pushed again from
// its slot (the same bits), then the wall and collision decisions.
template <int SP, int PPT>
__device__ __forceinline__ void step_deferred(CArgs& a, StepLds<PPT> S, uint64_t e, int qw,
                                              uint32_t ta0) {
  CSpecies& s = a.sp[SP];
  int64_t slot, dest;
  uint32_t births;
  step_place(S, e, qw, slot, dest, births);
  const bool cand = (((uint32_t)e >> 26) & 1u) != 0;
  const uint32_t id = (uint32_t)(e >> 32);
  double x = gptr(s.xin)[slot], vx = gptr(s.vxin)[slot];
  double vy = 0.0, vz = 0.0;
  if (cand || a.measuring) {
    const double2 pv = gptr(s.pv)[id];
    vy = pv.x;
    vz = pv.y;
  }
  int j;
  double f;
  int64_t w1;
  cell_of(x, a.inv_dx, a.nx, j, f, w1);
  push(S.E(), j, f, s.acc, s.dts, x, vx);
  const bool out = step_outside(a, x);
  uint32_t c = kCodePushed, o = 1u, b = 0u;
  step_need<SP, PPT>(a, S, dest, cand, x, vx, vy, vz, c, o, b);
  // a candidate inside the gap was stored and deposited as a plain output:
  // what its process changes is its code and, ionizing, one more output and a
  // birth
  const uint32_t had = out ? 0u : 1u;
  // (a null collision's code matters to nobody but a caller that records)
  if (c != (kCodePushed | (1u << 3)) || a.record) gptr(s.cout)[dest] = (uint8_t)c;
  step_tally<SP, PPT, true>(a, S, dest, ta0, o - 1u, b);
  if (o != had) {
    cell_of(x, a.inv_dx, a.nx, j, f, w1);
    const unsigned long long m = (unsigned long long)(o - had);
    atomicAdd(&S.H()[j], m * (unsigned long long)(kOne32 - w1));
    atomicAdd(&S.H()[j + 1], m * (unsigned long long)w1);
  }
  if (out) {
    gptr(s.xout)[dest] = x;
    gptr(s.vxout)[dest] = vx;
    gptr(s.idout)[dest] = id;
  }
}

// What a decision code implies for the outputs (outcome, as flags): bits 0-1
// outputs, bit 2 a birth, bit 3 queued, bit 4 the slot exists. A code of 0
// (slots taken as they are) is one plain output.
template <int SP>
__device__ __forceinline__ uint32_t step_flags(uint32_t c) {
  if (SP == 0) {
    if (c & 5u) return 16u;  // absorbed, or reflected past the other wall
    const uint32_t proc = (c >> 3) & 7u;
    return proc == 4u ? 16u | 8u | 4u | 2u : proc >= 2u ? 16u | 8u | 1u : 16u | 1u;
  }
  const uint32_t wall = c & 7u;
  if (wall) return wall == 3u ? 16u | 8u | 4u : 16u;
  return (c & kIonPending) ? 16u | 8u | 1u : 16u | 1u;
}

// The codes of the output slots [lo, lo + n) set to kCodePushed, four at a
// time where they are aligned: the code of every output until a wall, a
// process or an ion candidacy replaces it.
__device__ __forceinline__ void step_fill_codes(uint8_t* codes, uint32_t lo, uint32_t n) {
  constexpr uint32_t k4 = (uint32_t)kCodePushed * 0x01010101u;
  const uint32_t hi = lo + n;
  const uint32_t w0 = (lo + 3u) >> 2, w1 = hi >> 2;  // whole words
  if (w0 < w1) {
    uint32_t* w = reinterpret_cast<uint32_t*>(codes);
    for (uint32_t i = w0 + threadIdx.x; i < w1; i += kBlock) w[i] = k4;
    if (threadIdx.x < (w0 << 2) - lo) codes[lo + threadIdx.x] = kCodePushed;
    if (threadIdx.x < hi - (w1 << 2)) codes[(w1 << 2) + threadIdx.x] = kCodePushed;
  } else if (threadIdx.x < n) {
    codes[lo + threadIdx.x] = kCodePushed;  // fewer than seven
  }
}

// ---------------------------------------------------------------------------
// The tiles [t0, t1) of one species: prefO outputs and prefB births come
// before them. The field is in S.E; S.H and S.tally are zero on entry and on
// exit. Ends with a barrier.
//
// What bounds it is instructions and the registers that hold the waits, so
// everything uniform about a tile is uniform here: addresses are a tile's
// base plus a 32-bit lane offset, the default of every output (one plain
// particle: code, tile totals) is written for the tile as a whole, and only
// what differs is touched slot by slot.
template <int SP, int PPT, bool MEASURE, bool VAR>
__device__ __forceinline__ void step_tiles(CArgs& args, StepLds<PPT> S, int t0, int t1,
                                           int64_t n_tot, uint32_t prefO, uint32_t prefB) {
  using Tile = StepTile<PPT>;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const uint64_t lt = (1ull << lane) - 1ull;  // the lanes below this one
  const bool emit = args.sp[SP].emit != 0;
  const bool decide = args.sp[SP].decide != 0;
  const bool energy = MEASURE && SP == 0 && decide && args.measuring;
  const uint32_t ta0 = prefO / Tile::kSlots;
  int nq = 0, nd = 0;  // entries of this wave's queue
  int jr = -1;  // this lane's deposit run: cell jr, weights of nodes jr, jr + 1
  unsigned long long h0 = 0ull, h1 = 0ull;
  for (int t = t0;; ++t) {
    const bool fin = t >= t1;
    if (!fin) {
      const int p = (t - t0) & 1;
      const int ord = (t - t0) % kStepOrd;
      const uint32_t b0 = prefO >> 2;  // first draw block of the outputs
      uint32_t code[PPT], loc[Tile::kPairs], pid[PPT];
      double px[PPT], pvx[PPT], eps[MEASURE && SP == 0 ? PPT : 1];
      {
        CArgs& a = fresh(args);
        CSpecies& s = a.sp[SP];
        const int64_t base = (int64_t)t * Tile::kSlots;
        const uint32_t here = (uint32_t)min((int64_t)Tile::kSlots, n_tot - base);
        // (requested first: it is waited for before the particles)
        const uint32_t own_v = emit ? gptr(s.tin)[t] : here;
        const double* xi = gptr(s.xin) + base;
        const double* vi = gptr(s.vxin) + base;
        const uint32_t* ii = gptr(s.idin) + base;
        const uint8_t* ci = gptr(s.cin) + base;
        if (here == Tile::kSlots) {
#pragma unroll
          for (int k = 0; k < Tile::kPairs; ++k) {
            const uint32_t o = (uint32_t)(k * (2 * kBlock) + 2 * tid);
            const uint32_t c2 = emit ? (uint32_t)*reinterpret_cast<const uint16_t*>(ci + o) : 0u;
            const double2 xx = *reinterpret_cast<const double2*>(xi + o);
            const double2 vv = *reinterpret_cast<const double2*>(vi + o);
            const uint2 id = *reinterpret_cast<const uint2*>(ii + o);
            code[2 * k] = c2;
            px[2 * k] = xx.x;
            px[2 * k + 1] = xx.y;
            pvx[2 * k] = vv.x;
            pvx[2 * k + 1] = vv.y;
            pid[2 * k] = id.x;
            pid[2 * k + 1] = id.y;
          }
#pragma unroll
          for (int k = 0; k < Tile::kPairs; ++k) {
            const uint32_t c2 = code[2 * k];
            code[2 * k] = step_flags<SP>(c2 & 0xFFu) | ((c2 & 0x38u) << 5);
            code[2 * k + 1] = step_flags<SP>(c2 >> 8) | ((c2 >> 3) & 0x700u);
          }
        } else {
#pragma unroll
          for (int q = 0; q < PPT; ++q) {
            const uint32_t o = (uint32_t)((q >> 1) * (2 * kBlock) + 2 * tid + (q & 1));
            code[q] = 0u;
            px[q] = pvx[q] = 0.0;
            pid[q] = 0u;
            if (o < here) {
              const uint32_t c = emit ? (uint32_t)ci[o] : 0u;
              code[q] = step_flags<SP>(c) | ((c & 0x38u) << 5);  // the process from bit 8
              px[q] = xi[o];
              pvx[q] = vi[o];
              pid[q] = ii[o];
            }
          }
        }
        // the tile's outputs: their candidacy (one draw block of four slots
        // per thread), codes and totals, while the loads are in flight
        const uint32_t own = (uint32_t)uniform32((int)own_v) & 0xFFFFu;
        if (decide && own) {
          if (s.cand_thr) {
            const int nblk = (int)(((prefO + own - 1u) >> 2) - b0 + 1u);
            const uint64_t thr = s.cand_thr;
            for (int b = tid; b < nblk; b += kBlock) {
              const uint4 r = draw(a.dstep, b0 + (uint32_t)b, SP, 4, a.seed, a.run);
              S.s().cand[p][b] = (uint8_t)(((uint64_t)r.x < thr ? 1u : 0u) | ((uint64_t)r.y < thr ? 2u : 0u) |
                                           ((uint64_t)r.z < thr ? 4u : 0u) | ((uint64_t)r.w < thr ? 8u : 0u));
            }
          }
          const uint32_t room = (int64_t)prefO < s.cap ? (uint32_t)(s.cap - (int64_t)prefO) : 0u;
          const uint32_t n = min(own, room);
          step_fill_codes(gptr(s.cout), prefO, n);
          if (tid < 3) {
            // outputs [prefO, prefO + n) in output tile ta + tid
            const uint32_t ta = prefO / Tile::kSlots + (uint32_t)tid;
            const uint32_t lo = max(prefO, ta * Tile::kSlots);
            const uint32_t hi = min(prefO + n, (ta + 1u) * Tile::kSlots);
            if (hi > lo) step_tally<SP, PPT, true>(a, S, (int64_t)lo, ta0, hi - lo, 0u);
          }
        }
        if (energy) {
          // energy at the start of the decided step of an output that needs no
          // queued work
#pragma unroll
          for (int q = 0; q < PPT; ++q)
            if ((code[q] & 11u) == 1u) {
              const double2 pv = gptr(s.pv)[pid[q]];
              eps[MEASURE && SP == 0 ? q : 0] =
                  a.ek * (pvx[q] * pvx[q] + pv.x * pv.x + pv.y * pv.y);
            }
        }
      }
#pragma unroll
      for (int k = 0; k < Tile::kPairs; ++k) {
        const uint32_t c0 = code[2 * k], c1 = code[2 * k + 1];
        const uint32_t cnt = (c0 & 3u) + (c1 & 3u) + ((((c0 >> 2) & 1u) + ((c1 >> 2) & 1u)) << 16);
        const uint32_t inc = wave_incl_scan_dpp(cnt);
        loc[k] = inc - cnt;
        if (lane == kWave - 1) S.s().wtot[p][k][wave] = inc;
      }
      if (lane == 0) {
        uint32_t* pf = S.s().pref[wave][ord];
        pf[0] = prefO;
        pf[1] = prefB;
        pf[2] = (uint32_t)t;
      }
      __syncthreads();
      // every wave scans the tile's segment totals (segment k * waves + w)
      constexpr int nseg = Tile::kPairs * kStepWaves;
      const uint32_t sv = lane < nseg ? (&S.s().wtot[p][0][0])[lane] : 0u;
      const uint32_t si = wave_incl_scan_dpp(sv);
      const uint32_t tile_ob = (uint32_t)__builtin_amdgcn_readlane((int)si, nseg - 1);
      {
        CArgs& a = fresh(args);
        CSpecies& s = a.sp[SP];
        double* xo = gptr(s.xout) + prefO;
        double* vo = gptr(s.vxout) + prefO;
        uint32_t* io = gptr(s.idout) + prefO;
        uint8_t* co = gptr(s.cout) + prefO;
        const uint32_t room = (int64_t)prefO < s.cap ? (uint32_t)(s.cap - (int64_t)prefO) : 0u;
        const bool draws = decide && s.cand_thr != 0;
#pragma unroll
        for (int k = 0; k < Tile::kPairs; ++k) {
          uint32_t off =
              (uint32_t)__builtin_amdgcn_readlane((int)(si - sv), k * kStepWaves + wave) + loc[k];
          EnergyRun run{-1, 0.0, 0.0};
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int q = 2 * k + h;
            const uint32_t c = code[q];
            const uint32_t o = off & 0xFFFFu;
            const bool rare = (c & 8u) != 0;
            bool defer = false, cand = false;
            if ((c & 11u) == 1u && o < room) {
              double x = px[q], vx = pvx[q];
              bool keep = true;
              if (decide) {
                int jd;
                double fd;
                int64_t w1;
                cell_of(x, a.inv_dx, a.nx, jd, fd, w1);
                if (MEASURE && SP == 0) {
                  if (energy) step_energy(a, S, x, jd, w1, eps[MEASURE && SP == 0 ? q : 0], run);
                }
                push(S.E(), jd, fd, s.acc, s.dts, x, vx);
                if (draws) {
                  const uint32_t dest = prefO + o;
                  cand = ((S.s().cand[p][(dest >> 2) - b0] >> (dest & 3u)) & 1u) != 0;
                }
                keep = !step_outside(a, x);
                defer = !keep || (SP == 0 && cand);
                if (keep) {
                  if (SP == 1 && cand) {
                    // an ion candidate chooses its process when it is emitted
                    co[o] = (uint8_t)(kCodePushed | kIonPending);
                    atomicAdd(&S.s().cnt[C_I_CAND], 1ull);
                  }
                  cell_of(x, a.inv_dx, a.nx, jd, fd, w1);
                  if (jd != jr) {
                    if (jr >= 0) {
                      atomicAdd(&S.H()[jr], h0);
                      atomicAdd(&S.H()[jr + 1], h1);
                    }
                    jr = jd;
                    h0 = h1 = 0ull;
                  }
                  h0 += (unsigned long long)(kOne32 - w1);
                  h1 += (unsigned long long)w1;
                }
              }
              if (keep) {
                xo[o] = x;
                vo[o] = vx;
                io[o] = pid[q];
              }
            }
            // append to this wave's queue, in lane order
            const uint64_t mr = __ballot(rare), md = __ballot(defer);
            if (mr | md) {
              const uint32_t proc = SP == 0 ? c >> 8 : (c & 4u) ? kProcEmit : kProcIon;
              const uint64_t ent =
                  step_entry((uint32_t)(k * (2 * kWave) + 2 * lane + h), o, (uint32_t)ord, cand,
                             proc & 7u, rare && (c & 4u) ? off >> 16 : pid[q]);
              uint64_t* qu = S.s().q[wave];
              if (rare) qu[nq + __popcll(mr & lt)] = ent;
              if (defer) qu[Tile::kQueue - 1 - nd - __popcll(md & lt)] = ent;
              nq += __popcll(mr);
              nd += __popcll(md);
            }
            off += (c & 3u) + ((c & 4u) << 14);
          }
          if (MEASURE && SP == 0) step_energy_flush(S, run);
        }
      }
      prefO += tile_ob & 0xFFFFu;
      prefB += tile_ob >> 16;
    }
    // the queue: full waves of a kind, everything before an entry's tile
    // number is used again, and after the last tile what is left, shared by
    // the workgroup (one copy of this code: it is long)
    int np = 0, nr = 0;  // queued slots and deferred outputs to take
    int m[2][kStepWaves];
    if (!fin) {
      const bool drain = (t - t0) % kStepOrd == kStepOrd - 1;
      np = drain ? nq : nq & ~(kWave - 1);
      nr = drain ? nd : nd & ~(kWave - 1);
      if (np + nr == 0) continue;
      __threadfence_block();  // the queue, written by the other lanes
      nq -= np;
      nd -= nr;
    } else {
      if (lane == 0) {
        S.s().left[0][wave] = (uint32_t)nq;
        S.s().left[1][wave] = (uint32_t)nd;
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kStepWaves; ++w) {
        m[0][w] = uniform32((int)S.s().left[0][w]);
        m[1][w] = uniform32((int)S.s().left[1][w]);
        np += m[0][w];
        nr += m[1][w];
      }
    }
    const int step = fin ? kBlock : kWave;
    for (int i = fin ? tid : lane; i < np; i += step) {
      int w = fin ? 0 : wave, r = fin ? i : nq + i;
      if (fin) {
#pragma unroll
        for (int k = 0; k < kStepWaves - 1; ++k)
          if (w == k && r >= m[0][k]) {
            r -= m[0][k];
            ++w;
          }
      }
      step_queued<SP, PPT, MEASURE, VAR>(fresh(args), S, S.s().q[w][r], w, ta0);
    }
    for (int i = fin ? kBlock - 1 - tid : lane; i < nr; i += step) {
      int w = fin ? 0 : wave, r = fin ? i : nd + i;
      if (fin) {
#pragma unroll
        for (int k = 0; k < kStepWaves - 1; ++k)
          if (w == k && r >= m[1][k]) {
            r -= m[1][k];
            ++w;
          }
      }
      step_deferred<SP, PPT>(fresh(args), S, S.s().q[w][Tile::kQueue - 1 - r], w, ta0);
    }
    if (fin) break;
  }
  if (decide) {
    if (jr >= 0) {
      atomicAdd(&S.H()[jr], h0);
      atomicAdd(&S.H()[jr + 1], h1);
    }
    __syncthreads();
    CArgs& a = fresh(args);
    CSpecies& s = a.sp[SP];
    for (int j = tid; j < a.nx; j += kBlock) {
      const unsigned long long v = S.H()[j];
      if (v) {
        atomicAdd(&gptr(s.dep_out)[j], v);
        S.H()[j] = 0ull;
      }
    }
    if (tid < kStepTally) {
      const uint32_t v = S.s().tally[tid];
      if (v) {
        atomicAdd(&gptr(s.tout)[ta0 + (uint32_t)tid], v);
        S.s().tally[tid] = 0u;
      }
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// The tiles [u0, u1) of one discharge's sequence: te electron tiles, then ti
// ion tiles (at least one item, an empty one if the discharge has no
// particles). The workgroup that takes item 0 also writes the discharge's
// counts and, with self, its field.
template <int PPT, bool MEASURE, bool VAR>
__device__ __forceinline__ void step_segment(CArgs& a, StepLds<PPT> S, int u0, int u1,
                                             int te, int ti, int64_t ne, int64_t ni, bool zero_all) {
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = tid / kWave;
  const bool lead = u0 == 0;
  const bool emit_e = a.sp[0].emit != 0, emit_i = a.sp[1].emit != 0;
  const bool dec_e = a.sp[0].decide != 0, dec_i = a.sp[1].decide != 0;
  const int e1 = min(u1, te);
  const int i0 = max(u0, te) - te, i1 = u1 - te;  // this run's ion tiles

  // sums of both species' tile totals: all of them and those before this
  // workgroup's tiles (outputs, births)
  uint32_t v[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
  constexpr int kL = 4;
  if (emit_e) {
    for (int c0 = 0; c0 < te; c0 += kL * kBlock) {
      uint32_t w[kL];
#pragma unroll
      for (int k = 0; k < kL; ++k) {
        const int t = c0 + k * kBlock + tid;
        w[k] = t < te ? gptr(a.sp[0].tin)[t] : 0u;
      }
#pragma unroll
      for (int k = 0; k < kL; ++k) {
        const int t = c0 + k * kBlock + tid;
        v[0] += w[k] & 0xFFFFu;
        v[1] += w[k] >> 16;
        if (t < u0) {
          v[2] += w[k] & 0xFFFFu;
          v[3] += w[k] >> 16;
        }
      }
    }
  }
  if (emit_i) {
    for (int c0 = 0; c0 < ti; c0 += kL * kBlock) {
      uint32_t w[kL];
#pragma unroll
      for (int k = 0; k < kL; ++k) {
        const int t = c0 + k * kBlock + tid;
        w[k] = t < ti ? gptr(a.sp[1].tin)[t] : 0u;
      }
#pragma unroll
      for (int k = 0; k < kL; ++k) {
        const int t = c0 + k * kBlock + tid;
        v[4] += w[k] & 0xFFFFu;
        v[5] += w[k] >> 16;
        if (t < i0) {
          v[6] += w[k] & 0xFFFFu;
          v[7] += w[k] >> 16;
        }
      }
    }
  }
  if (dec_e) {
    if (a.self && a.nx <= kSelfSmallNx)
      step_field<kSelfSmallNx>(a, S.E(), S.s().w128, S.s().w64, lead);
    else if (a.self)
      step_field<kSelfMaxNx>(a, S.E(), S.s().w128, S.s().w64, lead);
    else
      stage_field<kBlock, 8>(S.E(), gptr(a.E), a.nx);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const uint32_t inc = wave_incl_scan_dpp(v[k]);
    if (lane == kWave - 1) S.s().red[k][wave] = inc;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    uint32_t t = 0u;
#pragma unroll
    for (int w = 0; w < kStepWaves; ++w) t += S.s().red[k][w];
    v[k] = (uint32_t)uniform32((int)t);
  }
  const uint32_t ae = emit_e ? v[0] : (uint32_t)min(ne, a.sp[0].cap);
  const int64_t ion0 = emit_i ? (int64_t)v[4] : ni;
  const int64_t pe = uniform64(gptr(a.pool_in)[0]), pi = uniform64(gptr(a.pool_in)[1]);
  if (tid == 0) {
    S.s().tot.ion0 = ion0;
    S.s().tot.se0 = (int64_t)ae;
    S.s().tot.pe = pe;
    S.s().tot.pi = pi;
    S.s().tot.pse = pe + (int64_t)v[1];
  }

  if (lead) {
    DevCtl* ctl = gptr(a.ctl);
    const int64_t ne2 = (int64_t)ae + (int64_t)v[5];
    const int64_t ni2 = ion0 + (int64_t)v[1];
    if (tid == 0) {
      if (emit_e) {
        ctl->n_e[a.par ^ 1] = ne2;
        ctl->n_i[a.par ^ 1] = ni2;
        const int64_t p0 = pe + (int64_t)v[1] + (int64_t)v[5], p1 = pi + (int64_t)v[1];
        gptr(a.pool_out)[0] = p0;
        gptr(a.pool_out)[1] = p1;
        if (ne2 > a.sp[0].cap || ni2 > a.sp[1].cap || p0 > a.sp[0].pcap || p1 > a.sp[1].pcap)
          latch_error(ctl, kErrCapacity);
      }
      if (dec_e) {
        const int64_t nd = min(emit_e ? ne2 : ne, a.sp[0].cap);
        count_add(ctl, C_E_PUSHED, (unsigned long long)nd);
        if (a.record) ctl->ncodes[0] = nd;
        const int64_t nid = min(emit_e ? ni2 : ni, a.sp[1].cap);
        if (dec_i) count_add(ctl, C_I_PUSHED, (unsigned long long)nid);
        ctl->ncodes[1] = dec_i && a.record ? nid : 0;
        if (a.self) {
          count_add(ctl, C_STEPS, 1ull);
          if (a.measuring) atomicAdd(reinterpret_cast<unsigned long long*>(&ctl->msteps), 1ull);
        }
      }
    }
    if (dec_e) {
      for (int j = tid; j < a.nx; j += kBlock) {
        gptr(a.sp[0].dep_zero)[j] = 0;
        gptr(a.sp[1].dep_zero)[j] = 0;
        if (!dec_i && !a.self)
          atomicAdd(&gptr(a.sp[1].dep_out)[j], (unsigned long long)gptr(a.sp[1].dep_in)[j]);
      }
      if (zero_all) {
#pragma unroll
        for (int sp = 0; sp < 2; ++sp)
          if (a.sp[sp].decide)
            for (int i = tid; i < a.sp[sp].ntz; i += kBlock) gptr(a.sp[sp].tzero)[i] = 0u;
      }
    }
  }

  if (u0 < e1) {
    const int64_t n = min(ne, a.sp[0].cap);
    step_tiles<0, PPT, MEASURE, VAR>(fresh(a), S, u0, e1, n,
                                     emit_e ? v[2] : (uint32_t)(u0 * StepTile<PPT>::kSlots),
                                     v[3]);
  }
  if (i0 < i1 && ti > 0) {
    const int64_t n = min(ni, a.sp[1].cap);
    step_tiles<1, PPT, MEASURE, VAR>(fresh(a), S, i0, min(i1, ti), n,
                                     emit_i ? v[6] : (uint32_t)(i0 * StepTile<PPT>::kSlots),
                                     v[7]);
  }
  // event counts and energy averages of this discharge
  if (tid < NCOUNTERS) {
    if (S.s().cnt[tid]) count_add(gptr(a.ctl), tid, S.s().cnt[tid]);
    S.s().cnt[tid] = 0ull;
  }
  if (MEASURE && a.measuring) {
    for (int j = tid; j < a.nx; j += kBlock) {
      const double e = S.EW()[j];
      if (e != 0.0) {
        atomicAdd(&gptr(a.acc_ew)[j], e);
        S.EW()[j] = 0.0;
      }
    }
    for (int b = tid; b < a.nbins; b += kBlock)
      if (S.EEPF()[b]) {
        atomicAdd(&gptr(a.eepf)[b], (unsigned long long)S.EEPF()[b]);
        S.EEPF()[b] = 0u;
      }
  }
}

// Particle counts and tiles of discharge a.
template <int PPT>
__device__ __forceinline__ void step_counts(CArgs& a, int64_t& ne, int64_t& ni, int& te, int& ti) {
  constexpr int kT = StepTile<PPT>::kSlots;
  ne = gptr(a.ctl)->n_e[a.par];
  ni = gptr(a.ctl)->n_i[a.par];
  te = (a.sp[0].emit || a.sp[0].decide) ? (int)((min(ne, a.sp[0].cap) + kT - 1) / kT) : 0;
  ti = (a.sp[1].emit || a.sp[1].decide) ? (int)((min(ni, a.sp[1].cap) + kT - 1) / kT) : 0;
}

// The number of items of a discharge's sequence that start below weight y:
// te electron tiles of weight we, then ti ion tiles of weight wi (one item of
// weight one if there are none).
__device__ __forceinline__ int step_items_below(int64_t y, int te, int ti, int we, int wi) {
  if (te + ti == 0) return y > 0 ? 1 : 0;
  const int64_t ye = (int64_t)te * we;
  if (y <= ye) return (int)((y + we - 1) / we);
  return te + (int)min((y - ye + wi - 1) / wi, (int64_t)ti);
}

// Clears the LDS a workgroup adds into.
template <int PPT, bool MEASURE>
__device__ __forceinline__ void step_clear(StepLds<PPT> S, int nx, int nbins) {
  const int tid = threadIdx.x;
  for (int j = tid; j < nx; j += kBlock) {
    S.H()[j] = 0ull;
    if (MEASURE) S.EW()[j] = 0.0;
  }
  if (MEASURE)
    for (int b = tid; b < nbins; b += kBlock) S.EEPF()[b] = 0u;
  if (tid < NCOUNTERS) S.s().cnt[tid] = 0ull;
  if (tid < kStepTally) S.s().tally[tid] = 0u;
}

template <int PPT, bool MEASURE, bool VAR>
__global__ __launch_bounds__(kBlock, step_min_waves(PPT, VAR)) void k_step(StepArgs) {
  CArgs& a = *(CArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  int64_t ne, ni;
  int te, ti;
  step_counts<PPT>(a, ne, ni, te, ti);
  ne = uniform64(ne);
  ni = uniform64(ni);
  te = uniform32(te);
  ti = uniform32(ti);
  if (a.sp[0].decide) {
#pragma unroll
    for (int sp = 0; sp < 2; ++sp)
      if (a.sp[sp].decide)
        for (int i = (int)blockIdx.x * kBlock + (int)threadIdx.x; i < a.sp[sp].ntz;
             i += (int)gridDim.x * kBlock)
          gptr(a.sp[sp].tzero)[i] = 0u;
  }
  // contiguous runs, the longer ones on the workgroups dispatched first
  const int n = max(te + ti, 1);
  const int g = (int)gridDim.x, b = (int)blockIdx.x;
  const int q = n / g, r = n % g;
  const int u0 = b < r ? b * (q + 1) : r * (q + 1) + (b - r) * q;
  const int u1 = u0 + (b < r ? q + 1 : q);
  if (u0 >= u1) return;
  const StepLds<PPT> S{a.nx};
  step_clear<PPT, MEASURE>(S, a.nx, a.nbins);
  __syncthreads();
  step_segment<PPT, MEASURE, VAR>(a, S, u0, u1, te, ti, ne, ni, false);
}

// A batch: workgroup b takes share k of g of discharge d (wgs[b]), by the
// weights of its tiles. The host deals the workgroups to the discharges, so
// that a workgroup needs only its own discharge's counts.
template <int PPT, bool MEASURE, bool VAR>
__global__ __launch_bounds__(kBlock, step_min_waves(PPT, VAR)) void k_step_b(
    const StepArgs* __restrict__ args, const StepWg* __restrict__ wgs, int nx_max, int nbins_max) {
  const __attribute__((address_space(4))) StepWg& w =
      ((const __attribute__((address_space(4))) StepWg*)(uintptr_t)wgs)[blockIdx.x];
  CArgs& a = ((CArgs*)(uintptr_t)args)[w.d];
  if (!a.sp[0].emit && !a.sp[0].decide) return;  // not part of this launch
  int64_t ne, ni;
  int te, ti;
  step_counts<PPT>(a, ne, ni, te, ti);
  ne = uniform64(ne);
  ni = uniform64(ni);
  te = uniform32(te);
  ti = uniform32(ti);
  const int we = a.sp[0].weight, wi = a.sp[1].weight;
  const int64_t load = max((int64_t)te * we + (int64_t)ti * wi, (int64_t)1);
  const int u0 = uniform32(step_items_below(load * w.k / w.g, te, ti, we, wi));
  const int u1 = uniform32(step_items_below(load * (w.k + 1) / w.g, te, ti, we, wi));
  if (u0 >= u1) return;
  const StepLds<PPT> S{nx_max};
  step_clear<PPT, MEASURE>(S, a.nx, a.nbins);
  __syncthreads();
  step_segment<PPT, MEASURE, VAR>(a, S, u0, u1, te, ti, ne, ni, true);
}

// ---------------------------------------------------------------------------
// host side

template <int PPT>
static size_t step_lds_bytes(int nx, int nbins, bool measure) {
  return sizeof(StepShared<PPT>) + (size_t)nx * 16 + (measure ? (size_t)nx * 8 + (size_t)nbins * 4 : 0);
}

// LDS is given out in steps of 160 KB / 128. The occupancy query divides by
// the exact size: between 1854 and 1907 points (not measuring) it promised
// three workgroups per CU where two fit, and the third of the grid that waited
// for a place ran alone (1900 cells, ions every 10th step, 4 million of each
// species: 74.7 us per step against 62.8).
constexpr size_t kLdsStep = 1280;

template <typename K>
static int step_blocks(K kern, size_t lds) {
  int nb = 0;
  lds = (lds + kLdsStep - 1) / kLdsStep * kLdsStep;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, kBlock, lds) != hipSuccess || nb < 1)
    nb = 1;
  return nb;
}

// The instance of (slots per thread, measuring, variants), one discharge's
// and the batch's: workgroups per CU that fit, or the launch.
template <int PPT, bool MEASURE, bool VAR>
struct StepInstance {
  static int fit(bool batch, int nx, int nbins) {
    const size_t lds = step_lds_bytes<PPT>(nx, nbins, MEASURE);
    return batch ? step_blocks(k_step_b<PPT, MEASURE, VAR>, lds)
                 : step_blocks(k_step<PPT, MEASURE, VAR>, lds);
  }
  static void one(const StepArgs& a, int grid, hipStream_t s) {
    hipLaunchKernelGGL((k_step<PPT, MEASURE, VAR>), dim3(grid), dim3(kBlock),
                       step_lds_bytes<PPT>(a.nx, a.nbins, MEASURE), s, a);
  }
  static void many(const StepArgs* args, const StepWg* wgs, int nx, int nbins, int grid,
                   hipStream_t s) {
    hipLaunchKernelGGL((k_step_b<PPT, MEASURE, VAR>), dim3(grid), dim3(kBlock),
                       step_lds_bytes<PPT>(nx, nbins, MEASURE), s, args, wgs, nx, nbins);
  }
};

// Calls f with the instance of the shape.
template <typename F>
static hipError_t step_instance(const StepShape& c, F f) {
  if (c.ppt == kStepPpt[0]) {
    if (c.measure)
      c.variants ? f(StepInstance<kStepPpt[0], true, true>()) : f(StepInstance<kStepPpt[0], true, false>());
    else
      c.variants ? f(StepInstance<kStepPpt[0], false, true>()) : f(StepInstance<kStepPpt[0], false, false>());
  } else if (c.ppt == kStepPpt[1]) {
    if (c.measure)
      c.variants ? f(StepInstance<kStepPpt[1], true, true>()) : f(StepInstance<kStepPpt[1], true, false>());
    else
      c.variants ? f(StepInstance<kStepPpt[1], false, true>()) : f(StepInstance<kStepPpt[1], false, false>());
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t step_fit(StepShape& c, bool batch, int nx, int nbins) {
  return step_instance(c, [&](auto k) { c.fit = decltype(k)::fit(batch, nx, nbins); });
}

void step_grid(StepShape& c, int num_cu, int wg_per_cu, int64_t max_tiles) {
  const int nb = wg_per_cu > 0 && c.fit > wg_per_cu ? wg_per_cu : c.fit;
  int64_t g = (int64_t)nb * num_cu;
  if (g > max_tiles) g = max_tiles;
  c.grid = g < 1 ? 1 : (int)g;
}

hipError_t launch_step_kernel(const StepArgs& a, const StepShape& c, hipStream_t s) {
  if (a.nx > kMaxNx || a.nx < 3 || (a.self && a.nx > kSelfMaxNx) || c.grid < 1)
    return hipErrorInvalidValue;
  return step_instance(c, [&](auto k) { decltype(k)::one(a, c.grid, s); });
}

hipError_t launch_step_batch(const StepArgs* args, const StepWg* wgs, const StepShape& c,
                             int nx_max, int nbins_max, hipStream_t s) {
  if (nx_max > kMaxNx || nx_max < 3 || c.grid < 1) return hipErrorInvalidValue;
  return step_instance(c,
                       [&](auto k) { decltype(k)::many(args, wgs, nx_max, nbins_max, c.grid, s); });
}

}  // namespace pic
