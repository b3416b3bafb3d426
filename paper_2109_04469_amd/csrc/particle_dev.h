// Device functions of the particle passes shared by the per-pass kernels
// (k_particle.hip) and the one-kernel step (k_step.hip): gather and push,
// decision codes, deposits, collision kinematics and emission
// (arXiv:2109.04469, Sec. 2 steps 3-6).
#pragma once

#include "pic_internal.h"

namespace pic {

// Copies a field of nx values into LDS, PER loads of each thread issued
// before its first store (one memory round trip per PER strides of the
// workgroup instead of one per stride).
template <int NT, int PER>
__device__ __forceinline__ void stage_field(double* sE, const double* E, int nx) {
  for (int j0 = (int)threadIdx.x; j0 < nx; j0 += PER * NT) {
    double v[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int j = j0 + k * NT;
      v[k] = j < nx ? E[j] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int j = j0 + k * NT;
      if (j < nx) sE[j] = v[k];
    }
  }
}

// Code bit used between the kernels of a pass only: an Ar+ collision
// candidate whose process (which needs a thermal atom velocity) is chosen by
// the kernel that takes the queued slots, which replaces it with the process
// bits, so a code read by the caller has bit 6 clear.
constexpr uint32_t kIonPending = 0x40u;

struct Outcome {
  uint32_t own;    // output slots of this species: 0, 1 or 2
  uint32_t birth;  // births of the other species: 0 or 1
  bool rare;       // queued: needs draws (collision kinematics, an emission)
};

// What a decision code implies for the outputs. Slots carried without a
// push (bit 7 clear) give one output.
template <int SP>
__device__ __forceinline__ Outcome outcome(uint32_t c) {
  Outcome r{0u, 0u, false};
  if (!(c & kCodePushed)) {
    r.own = 1u;
    return r;
  }
  const uint32_t wall = c & 7u;
  const uint32_t proc = (c >> 3) & 7u;
  if (SP == 0) {
    const bool alive = wall == 0u || wall == 2u;
    const bool ion = alive && proc == 4u;
    r.own = alive ? (ion ? 2u : 1u) : 0u;
    r.birth = ion ? 1u : 0u;
    r.rare = alive && proc >= 2u;
  } else {
    const bool alive = wall == 0u;
    r.own = alive ? 1u : 0u;
    r.birth = wall == 3u ? 1u : 0u;
    r.rare = (alive && (c & kIonPending)) || wall == 3u;
  }
  return r;
}

// Gather (linear interpolation in the particle's cell) and leap-frog push.
// Every kernel calls this on the same inputs and gets the same bits.
__device__ __forceinline__ void push(const double* E, int j, double f, double acc, double dts,
                                     double& x, double& vx) {
  const double Ep = (1.0 - f) * E[j] + f * E[j + 1];
  vx = vx + acc * Ep;
  x = x + vx * dts;
}


__device__ __forceinline__ void deposit_global(unsigned long long* dep, double x, double inv_dx,
                                               int nx) {
  int j;
  double f;
  int64_t w1;
  cell_of(x, inv_dx, nx, j, f, w1);
  atomicAdd(&dep[j], (unsigned long long)(kOne32 - w1));
  atomicAdd(&dep[j + 1], (unsigned long long)w1);
}

// Cumulative collision frequency of process `p` of NP at table variable tv
// (speed / table step), linear in tv; beyond the last table speed, the last
// entry. The processes of one speed lie next to each other, so a candidate's
// reads share one or two cache lines.
template <int NP>
__device__ __forceinline__ double cum_nu(const double* cum, int ntab, int p, double tv) {
  if (tv < (double)(ntab - 1)) {
    const int kk = (int)tv;
    const double tt = tv - (double)kk;
    const double* c = cum + (int64_t)kk * NP + p;
    return (1.0 - tt) * c[0] + tt * c[NP];
  }
  return cum[(int64_t)(ntab - 1) * NP + p];
}

// Direction after a deflection by chi from the incident unit vector e, with
// cos chi = (2 + eps - 2 (1 + eps)^u) / eps (eps in eV; uniform cos chi when
// eps = 0) and azimuth 2 pi w, about e: n = cos chi e + sin chi (cos phi b1 +
// sin phi b2), b1 the unit vector along e x (1, 0, 0) (e x (0, 1, 0) when e
// is within 26 degrees of the x axis), b2 = e x b1.
__device__ __forceinline__ void aniso_dir(double ex, double ey, double ez, double eps, double u,
                                          double w, double& nx, double& ny, double& nz) {
  double c = eps > 0.0 ? (2.0 + eps - 2.0 * pow(1.0 + eps, u)) / eps : 1.0 - 2.0 * u;
  c = fmin(fmax(c, -1.0), 1.0);
  const double sn = sqrt(fmax(1.0 - c * c, 0.0));
  const double ph = kTwoPi * w;
  double sp, cp;
  sincos(ph, &sp, &cp);
  double b1x, b1y, b1z;
  if (fabs(ex) < 0.9) {  // e x (1, 0, 0) = (0, ez, -ey)
    const double r = sqrt(ey * ey + ez * ez);
    b1x = 0.0;
    b1y = ez / r;
    b1z = -ey / r;
  } else {  // e x (0, 1, 0) = (-ez, 0, ex)
    const double r = sqrt(ez * ez + ex * ex);
    b1x = -ez / r;
    b1y = 0.0;
    b1z = ex / r;
  }
  const double b2x = ey * b1z - ez * b1y;
  const double b2y = ez * b1x - ex * b1z;
  const double b2z = ex * b1y - ey * b1x;
  nx = c * ex + sn * (cp * b1x + sp * b2x);
  ny = c * ey + sn * (cp * b1y + sp * b2y);
  nz = c * ez + sn * (cp * b1z + sp * b2z);
}

// Velocities after a collision of an electron (the draws of slot `slot` at
// step `step`): proc 2 elastic, 3 excitation, 4 ionization, which also makes
// a second electron (velocity cv) and a thermal ion (velocity bv) and returns
// true. VAR: the method-variant paths (anisotropic elastic scattering, Opal
// sharing) are compiled in; without them the kernels stay smaller. A: an
// argument block with the collision constants.
template <bool VAR, class A>
__device__ __forceinline__ bool electron_collision(const A& a, uint32_t step, uint32_t slot,
                                                   uint32_t proc, double& vx, double& vy,
                                                   double& vz, double* cv, double* bv) {
  const uint4 r1 = draw(step, slot, 0, 1, a.seed, a.run);
  const double v2 = vx * vx + vy * vy + vz * vz;
  const bool elastic = proc == 2, ionize = proc == 4;
  // the three processes share their square root and direction (lanes of
  // different processes do not take turns there)
  double e_ej = 0.0, arg = v2;
  if (!elastic) {
    // the threshold energy is lost; an ionization shares the rest uniformly,
    // or (variant) as Opal et al.
    double eps = a.ek * v2 - (ionize ? a.ion_thr : a.exc_thr);
    if (eps < 0.0) eps = 0.0;
    if (ionize) {
      const uint4 r2 = draw(step, slot, 0, 2, a.seed, a.run);
      e_ej = (VAR && (a.model & kModelOpal))
                 ? kOpalW * tan(u01(r2.x) * atan(eps / (2.0 * kOpalW)))
                 : u01(r2.x) * eps;
      eps = eps - e_ej;
    }
    arg = eps * a.ve;
  }
  const double speed = sqrt(arg);
  double nx_, ny_, nz_;
  if (VAR && elastic && (a.model & kModelAniso) && speed > 0.0)
    aniso_dir(vx / speed, vy / speed, vz / speed, a.ek * v2, u01(r1.x), u01(r1.y), nx_, ny_, nz_);
  else
    iso_dir(u01(r1.x), u01(r1.y), nx_, ny_, nz_);
  if (elastic) {
    // on an atom at rest: isotropic in the CM frame, or (variant) deflected
    // by the screened-Coulomb angle about the incident direction
    const double gg = a.mm * speed;
    vx = a.mr * vx + gg * nx_;
    vy = a.mr * vy + gg * ny_;
    vz = a.mr * vz + gg * nz_;
    return false;
  }
  vx = speed * nx_;
  vy = speed * ny_;
  vz = speed * nz_;
  if (!ionize) return false;
  // the second electron, isotropic, and the new ion, thermal
  const uint4 r3 = draw(step, slot, 0, 3, a.seed, a.run);
  const double s_ej = sqrt(e_ej * a.ve);
  double bx, by, bz;
  iso_dir(u01(r1.z), u01(r1.w), bx, by, bz);
  cv[0] = s_ej * bx;
  cv[1] = s_ej * by;
  cv[2] = s_ej * bz;
  double n1, n2, n3, dmy;
  box_muller(u01(r3.x), u01(r3.y), n1, n2);
  box_muller(u01(r3.z), u01(r3.w), n3, dmy);
  bv[0] = a.sig_g * n1;
  bv[1] = a.sig_g * n2;
  bv[2] = a.sig_g * n3;
  return true;
}

// An Ar+ candidate on a thermal atom drawn for it: isotropic elastic in the
// CM frame (returns 2), backward (charge transfer, 3), or null (1). beyond:
// its relative speed lies past the last table entry.
template <class A>
__device__ __forceinline__ uint32_t ion_collision(const A& a, uint32_t step, uint32_t slot,
                                                  const double* cum, double numax, double inv_dv,
                                                  double& vx, double& vy, double& vz,
                                                  bool& beyond) {
  const uint4 r0 = draw(step, slot, 1, 0, a.seed, a.run);
  const uint4 r1 = draw(step, slot, 1, 1, a.seed, a.run);
  double n1, n2, n3, dmy;
  box_muller(u01(r1.x), u01(r1.y), n1, n2);
  box_muller(u01(r1.z), u01(r1.w), n3, dmy);
  const double ax = a.sig_g * n1, ay = a.sig_g * n2, az = a.sig_g * n3;
  const double gx = vx - ax, gy = vy - ay, gz = vz - az;
  const double g = sqrt(gx * gx + gy * gy + gz * gz);
  const double tv = g * inv_dv;
  beyond = !(tv < (double)(a.ntab - 1));
  const double r = u01(r0.z) * numax;
  const double c0 = cum_nu<2>(cum, a.ntab, 0, tv), c1 = cum_nu<2>(cum, a.ntab, 1, tv);
  if (r < c0) {
    const uint4 r2 = draw(step, slot, 1, 2, a.seed, a.run);
    double ux, uy, uz;
    iso_dir(u01(r2.x), u01(r2.y), ux, uy, uz);
    const double hg = 0.5 * g;
    vx = 0.5 * (vx + ax) + hg * ux;
    vy = 0.5 * (vy + ay) + hg * uy;
    vz = 0.5 * (vz + az) + hg * uz;
    return 2u;
  }
  if (r < c1) {
    vx = ax;
    vy = ay;
    vz = az;
    return 3u;
  }
  return 1u;
}

// Secondary electron of the ion in `slot`, which left the gap at x:
// half-Maxwellian from the wall it hit. bx: the wall's position.
template <class A>
__device__ __forceinline__ void secondary_electron(const A& a, uint32_t step, uint32_t slot,
                                                   double x, double& bx, double* bv) {
  const uint4 r3 = draw(step, slot, 1, 3, a.seed, a.run);
  double n1, n2, n3, dmy;
  box_muller(u01(r3.x), u01(r3.y), n1, n2);
  box_muller(u01(r3.z), u01(r3.w), n3, dmy);
  bx = (x < 0.0) ? 0.0 : a.L;
  bv[0] = a.sig_se * fabs(n1);
  if (x > a.L) bv[0] = -bv[0];
  bv[1] = a.sig_se * n2;
  bv[2] = a.sig_se * n3;
}

}  // namespace pic
