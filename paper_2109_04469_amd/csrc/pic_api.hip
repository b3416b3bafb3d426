// libpic C ABI: parameter validation, derived constants, workspace layout
// and the per-step launch schedule. Host code only; every step of the method
// runs in the kernels of k_field / k_particle / k_sort.
#include <cmath>
#include <cstddef>
#include <cstdio>
#include <cstring>
#include <new>
#include <queue>
#include <vector>

#include "../../include/warmstart.h"
#include "pic_internal.h"

using namespace pic;

struct pic_batch {
  std::vector<pic_handle*> hs;
  hipStream_t stream;
  int num_cu;
  int nx_max, nbins_max;
  bool variants;      // some discharge uses a method variant
  int chunk;          // steps per upload of argument blocks
  unsigned char* dev[2];
  unsigned char* host[2];
  hipEvent_t copied[2];
  int slot;
  int64_t* counts;  // pinned, per discharge: electrons, ions after `chunk` steps
  int64_t unseen;   // steps since the counts were asked for
  int step_fit[2][2];  // one-kernel steps' workgroups per CU, per tile size and measuring
  BatchLaunch passes;  // launches of the passes
};

namespace {

constexpr size_t kAlign = 256;
constexpr int kMaxCells = 4096;

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// Velocity-pool entries per buffer: the live particles plus the entries of
// particles absorbed and born since the last repack (every sort, or every
// kRepackSteps steps when sorts are rarer). Running out latches
// PIC_ECAPACITY.
constexpr int kRepackSteps = 256;
int64_t pool_capacity(int64_t cap) { return cap + (cap / 2 > 4096 ? cap / 2 : 4096); }

// Upper edge of the ion arrival-energy bins: ions gain at most about the
// peak sheath voltage, so 1.25 phi_0 (at least 10 eV).
double fedf_ion_emax(double rf_voltage_v) {
  const double e = 1.25 * rf_voltage_v;
  return e > 10.0 ? e : 10.0;
}

struct Layout {
  size_t ctl, part[2][2][2], pid[2][2], pool[2][2], codes[2][2], tcnt[2][2], rq[2], stc[2][3], dep[2][3], rho, phi, E[2], cum[2], th_cp,
      th_m, acc_ne, acc_ni, acc_w, acc_ew, eepf, fedf[2], sort_cnt[2], sort_tot[2], cand, dq, total;
  int64_t max_tiles[2];
  int64_t stc_n[2];
  int sort_blocks;
};

int validate(const pic_params* p, const pic_xsec* xs) {
  if (!p || !xs) return PIC_EINVAL;
  if (!(p->gap_m > 0) || !(p->rf_freq_hz > 0) || p->steps_per_cycle < 1) return PIC_EINVAL;
  if (p->n_cells < 2 || p->n_cells > kMaxCells) return PIC_EINVAL;
  if (!(p->weight > 0) || !(p->area_m2 > 0) || !(p->gas_temp_k > 0) || !(p->pressure_pa >= 0))
    return PIC_EINVAL;
  if (!(p->reflection >= 0 && p->reflection <= 1) || !(p->gamma_see >= 0 && p->gamma_see <= 1))
    return PIC_EINVAL;
  if (!(p->see_temp_ev >= 0)) return PIC_EINVAL;
  for (int s = 0; s < 2; ++s)
    if (p->capacity[s] < 0 || p->capacity[s] > ((int64_t)1 << 31) - kTile) return PIC_EINVAL;
  if (p->ion_subcycle < 1 || p->sort_interval < 0) return PIC_EINVAL;
  if (p->eepf_bins < 1 || p->eepf_bins > 4096 || !(p->eepf_emax_ev > 0) ||
      !(p->eepf_halfwidth_m >= 0))
    return PIC_EINVAL;
  if (xs->n < 2 || !(xs->dv_e > 0) || !(xs->dv_i > 0)) return PIC_EINVAL;
  for (int k = 0; k < 3; ++k)
    if (!xs->sigma_e[k]) return PIC_EINVAL;
  for (int k = 0; k < 2; ++k)
    if (!xs->sigma_i[k]) return PIC_EINVAL;
  if (!(xs->exc_threshold_ev >= 0) || !(xs->ion_threshold_ev >= 0)) return PIC_EINVAL;
  const uint32_t known = PIC_FLAG_NO_FIELD | PIC_FLAG_FIXED_E | PIC_FLAG_NO_COLL |
                         PIC_FLAG_IMMOBILE_IONS | PIC_FLAG_RECORD | PIC_FLAG_THOMAS |
                         PIC_FLAG_ANISO_ELASTIC | PIC_FLAG_OPAL_SHARING;
  if (p->flags & ~known) return PIC_EINVAL;
  return PIC_OK;
}

Layout make_layout(const pic_params* p, const pic_xsec* xs) {
  Layout L{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off += align_up(bytes > 0 ? bytes : 1);
    return o;
  };
  const int nx = p->n_cells + 1;
  L.ctl = take(sizeof(DevCtl));
  for (int s = 0; s < 2; ++s) {
    const int64_t cap = p->capacity[s];
    L.max_tiles[s] = (cap + kTile - 1) / kTile + 1;
    for (int b = 0; b < 2; ++b) {
      for (int q = 0; q < 2; ++q) L.part[s][b][q] = take((size_t)cap * sizeof(double));
      L.pid[s][b] = take((size_t)cap * sizeof(uint32_t));
      L.pool[s][b] = take((size_t)pool_capacity(cap) * sizeof(double2));
    }
    for (int b = 0; b < 2; ++b) L.codes[s][b] = take((size_t)cap);
    for (int b = 0; b < 2; ++b) L.tcnt[s][b] = take((size_t)L.max_tiles[s] * sizeof(uint64_t));
    L.rq[s] = take((size_t)cap * 16);
    L.stc_n[s] = (cap + kStepMinTile - 1) / kStepMinTile + 1;
    for (int b = 0; b < 3; ++b) L.stc[s][b] = take((size_t)L.stc_n[s] * sizeof(uint32_t));
    for (int b = 0; b < 3; ++b) L.dep[s][b] = take((size_t)nx * 8);
  }
  L.rho = take((size_t)nx * 8);
  L.phi = take((size_t)nx * 8);
  for (int b = 0; b < 2; ++b) L.E[b] = take((size_t)nx * 8);
  L.cum[0] = take((size_t)3 * xs->n * 8);
  L.cum[1] = take((size_t)2 * xs->n * 8);
  L.th_cp = take((size_t)nx * 8);
  L.th_m = take((size_t)nx * 8);
  L.acc_ne = take((size_t)nx * 8);
  L.acc_ni = take((size_t)nx * 8);
  L.acc_w = take((size_t)nx * 8);
  L.acc_ew = take((size_t)nx * 8);
  L.eepf = take((size_t)p->eepf_bins * 8);
  for (int sp = 0; sp < 2; ++sp) L.fedf[sp] = take((size_t)2 * p->eepf_bins * 8);
  int64_t capmax = p->capacity[0] > p->capacity[1] ? p->capacity[0] : p->capacity[1];
  int sb = (int)((capmax + 4095) / 4096);
  if (sb < 1) sb = 1;
  if (sb > kMaxSortBlocks) sb = kMaxSortBlocks;
  L.sort_blocks = sb;
  for (int s = 0; s < 2; ++s) {
    L.sort_cnt[s] = take((size_t)sb * (size_t)(nx - 1) * sizeof(uint32_t));
    L.sort_tot[s] = take((size_t)(nx - 1) * sizeof(uint32_t));
  }
  // candidacy bits of the electron slots of a pipelined step
  L.cand = take((size_t)((p->capacity[0] + 31) / 32 + 1) * sizeof(uint32_t));
  L.dq = take((size_t)p->capacity[0] * sizeof(uint32_t));
  L.total = off;
  return L;
}

// u01(r) = (r + 1/2) 2^-32 is exact in FP64, so u01(r) < p holds exactly
// when r + 1/2 < P = p 2^32 (scaling by a power of two is exact), i.e. for
// integers r < ceil(P - 1/2); P - 1/2 is exact for P < 2^32.
uint64_t candidacy_threshold(double p) {
  if (!(p > 0.0)) return 0;
  if (p >= 1.0) return (uint64_t)1 << 32;
  const double t = std::ceil(std::ldexp(p, 32) - 0.5);
  return t <= 0.0 ? 0 : (uint64_t)t;
}

int hip_status(hipError_t e) { return e == hipSuccess ? PIC_OK : PIC_EHIP; }

#define HIP_TRY(expr)                        \
  do {                                       \
    hipError_t _e = (expr);                  \
    if (_e != hipSuccess) return PIC_EHIP;   \
  } while (0)

// Starts a timed launch: returns the event index or -1 when timing is off.
int timer_begin(pic_handle* h) {
  if (!h->timing) return -1;
  const size_t need = 2 * (h->ev_next + 1);
  while (h->ev_pool.size() < need) {
    hipEvent_t e;
    // timing-only events: no system-scope fence (no cache writeback) on record
    if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) return -1;
    h->ev_pool.push_back(e);
  }
  const int idx = (int)(2 * h->ev_next);
  if (hipEventRecord(h->ev_pool[idx], h->stream) != hipSuccess) return -1;
  h->ev_next += 1;
  return idx;
}

void timer_end(pic_handle* h, int timer, int idx) {
  if (idx < 0) return;
  if (hipEventRecord(h->ev_pool[idx + 1], h->stream) == hipSuccess)
    h->ev_used.emplace_back(timer, idx);
}

// Folds the recorded event pairs into the per-timer sums (synchronises).
int timer_collect(pic_handle* h) {
  if (h->ev_used.empty()) {
    h->ev_next = 0;
    return PIC_OK;
  }
  if (hipStreamSynchronize(h->stream) != hipSuccess) return PIC_EHIP;
  for (const auto& u : h->ev_used) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, h->ev_pool[u.second], h->ev_pool[u.second + 1]) != hipSuccess)
      return PIC_EHIP;
    h->t_ms[u.first] += ms;
    h->t_n[u.first] += 1;
  }
  h->ev_used.clear();
  h->ev_next = 0;
  return PIC_OK;
}

// ---- reading calls: one kernel writes what they need to pinned host memory,
// one wait for the stream

size_t report_words(const pic_handle* h) {
  const size_t nx = (size_t)h->nx, nb = (size_t)h->p.eepf_bins;
  const size_t a = 5 * nx + nb, b = 4 * nb;
  return R_ARRAYS + (a > b ? a : b);
}

ReportArgs report_args(const pic_handle* h) {
  ReportArgs a{};
  a.ctl = h->ctl;
  a.out = h->report;
  a.par = (int)(h->step & 1);
  return a;
}

// The host has seen the particle count of a species; it waited for the stream
// then, so a count from an earlier step is no news any more.
void saw_count(pic_handle* h, int sp, int64_t n) {
  h->hint[sp] = n < h->p.capacity[sp] ? n : h->p.capacity[sp];
  h->hint_new = 1;
  h->seen[sp] = -1;
}

int report_status(const pic_handle* h) {
  const uint64_t err = h->report[R_ERR];
  if (err & kErrUnstable) return PIC_EUNSTABLE;
  if (err & kErrCapacity) return PIC_ECAPACITY;
  return PIC_OK;
}

// Reads the report of a into h->report; PIC_EHIP if that failed.
int read_report(pic_handle* h, const ReportArgs& a) {
  HIP_TRY(launch_report(a, h->stream));
  HIP_TRY(hipStreamSynchronize(h->stream));
  for (int s = 0; s < 2; ++s) saw_count(h, s, (int64_t)h->report[s == 0 ? R_NE : R_NI]);
  h->unseen = 0;
  return PIC_OK;
}

// Waits for the stream and returns the first latched device error, if any.
int latched(pic_handle* h) {
  const int st = read_report(h, report_args(h));
  return st ? st : report_status(h);
}

// Memory of the handle's own GPU.
bool on_device(const pic_handle* h, const void* p) {
  hipPointerAttribute_t at;
  if (hipPointerGetAttributes(&at, p) != hipSuccess) {
    (void)hipGetLastError();  // unknown memory: the caller's own host memory
    return false;
  }
  return at.type == hipMemoryTypeDevice && at.device == h->device && (uintptr_t)p % 8 == 0;
}

// Memory the host may write: its own or pinned. Anything else (a device
// array, also a misaligned one or another GPU's; managed memory) takes a copy.
bool on_host(const void* p) {
  hipPointerAttribute_t at;
  if (hipPointerGetAttributes(&at, p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return at.type == hipMemoryTypeUnregistered || at.type == hipMemoryTypeHost;
}

int field_mode(const pic_handle* h) {
  const uint32_t f = h->p.flags;
  if (f & PIC_FLAG_NO_FIELD) return FIELD_ZERO;
  if (f & PIC_FLAG_FIXED_E) return FIELD_FIXED;
  if (f & PIC_FLAG_THOMAS) return FIELD_THOMAS;
  return FIELD_EXACT;
}

// The species' deposit buffer `ahead` places after the current one.
int64_t* dep_buf(const pic_handle* h, int sp, int ahead) {
  return h->dep[sp][(h->dsel[sp] + ahead) % 3];
}

int64_t* pool_levels(const pic_handle* h) { return h->ctl->pool_n[h->psel]; }

PartArgs particle_args(pic_handle* h, int sp, int parity) {
  PartArgs a{};
  const int in = h->cur[sp], out = 1 - h->cur[sp];
  a.xin = h->part[sp][in][0];
  a.vxin = h->part[sp][in][1];
  a.idin = h->pid[sp][in];
  a.xout = h->part[sp][out][0];
  a.vxout = h->part[sp][out][1];
  a.idout = h->pid[sp][out];
  a.pv = h->pool[sp][h->pcur[sp]];
  a.pcap = h->pcap[sp];
  const int other = 1 - sp;
  // electrons append ions to the current ion buffer; ions append secondary
  // electrons to the electron buffer the electron kernel has just written
  const int ob = h->cur[other];
  a.bx = h->part[other][ob][0];
  a.bvx = h->part[other][ob][1];
  a.bid = h->pid[other][ob];
  a.bpv = h->pool[other][h->pcur[other]];
  a.bpcap = h->pcap[other];
  a.E = h->Ebuf[parity];
  if (sp == 0) {
    a.dep_own = reinterpret_cast<unsigned long long*>(dep_buf(h, 0, 1));
    a.dep_other = reinterpret_cast<unsigned long long*>(dep_buf(h, 1, 0));
  } else {
    a.dep_own = reinterpret_cast<unsigned long long*>(dep_buf(h, 1, 1));
    a.dep_other = reinterpret_cast<unsigned long long*>(dep_buf(h, 0, 1));
  }
  a.cum = h->cum[sp];
  a.ctl = h->ctl;
  a.pool_n = pool_levels(h);
  // tile totals are summed with atomics into a buffer the previous pass of
  // this species zeroed; this pass zeroes the other one
  a.tcnt = h->tcnt[sp][h->tsel[sp]];
  a.tcnt_next = h->tcnt[sp][h->tsel[sp] ^ 1];
  a.rq = h->rq[sp];
  // decision codes of alternate passes in alternate buffers: a pass fused
  // with the next step's decisions reads one and writes the other
  a.codes = h->codes[sp][h->csel[sp]];
  a.cand = sp == 0 ? h->cand : nullptr;
  a.dq = sp == 0 ? h->dq : nullptr;
  a.acc_ew = h->acc_ew;
  a.eepf = h->eepf;
  a.fedf = h->fedf[sp];
  a.ek_s = 0.5 * h->mass[sp] / kQe;
  a.fedf_inv_de = (double)h->p.eepf_bins / h->fedf_emax[sp];
  a.measure_walls = h->measuring;
  a.cap = h->p.capacity[sp];
  a.bcap = h->p.capacity[other];
  a.max_tiles = h->max_tiles[sp];
  a.inv_dx = h->inv_dx;
  a.L = h->L;
  a.acc = h->acc[sp];
  a.dts = h->dts[sp];
  a.p_wall = sp == 0 ? h->p.reflection : h->p.gamma_see;
  a.pcoll = h->pcoll[sp];
  a.pcoll_thr = candidacy_threshold(h->pcoll[sp]);
  a.numax = h->numax[sp];
  a.inv_dv = h->inv_dv[sp];
  a.mr = h->mr_e;
  a.mm = h->mm_e;
  a.ek = h->ek_e;
  a.ve = h->ve_e;
  a.exc_thr = h->exc_thr;
  a.ion_thr = h->ion_thr;
  a.sig_g = h->sig_g;
  a.sig_se = h->sig_se;
  a.half = 0.5 * h->L;
  a.eepf_hw = h->p.eepf_halfwidth_m;
  a.inv_de = h->inv_de;
  a.nx = h->nx;
  a.ntab = h->ntab;
  a.nbins = h->p.eepf_bins;
  a.parity = parity;
  a.step = (uint32_t)h->step;
  a.seed = h->p.seed;
  a.run = h->p.run;
  a.no_coll = (h->p.flags & PIC_FLAG_NO_COLL) ? 1 : 0;
  a.record = (h->p.flags & PIC_FLAG_RECORD) ? 1 : 0;
  a.model = ((h->p.flags & PIC_FLAG_ANISO_ELASTIC) ? kModelAniso : 0) |
            ((h->p.flags & PIC_FLAG_OPAL_SHARING) ? kModelOpal : 0);
  return a;
}

SortArgs sort_args(pic_handle* h, int sp, bool reorder) {
  SortArgs a{};
  const int in = h->cur[sp], out = reorder ? 1 - h->cur[sp] : h->cur[sp];
  const int pin = h->pcur[sp], pout = 1 - h->pcur[sp];
  a.sx = h->part[sp][in][0];
  a.svx = h->part[sp][in][1];
  a.sid = h->pid[sp][in];
  a.spv = h->pool[sp][pin];
  a.dx = h->part[sp][out][0];
  a.dvx = h->part[sp][out][1];
  a.did = h->pid[sp][out];
  a.dpv = h->pool[sp][pout];
  a.pool_n = &pool_levels(h)[sp];
  a.count = sp == 0 ? &h->ctl->n_e[h->step & 1] : &h->ctl->n_i[h->step & 1];
  a.cap = h->p.capacity[sp];
  a.cnt = h->sort_cnt[sp];
  a.tot = h->sort_tot[sp];
  a.inv_dx = h->inv_dx;
  a.nx = h->nx;
  a.hint = h->hint[sp];
  a.nblocks = h->sort_blocks;
  return a;
}

FieldArgs field_args(pic_handle* h, int field_mode_, bool ion_step) {
  const int par = (int)(h->step & 1);
  FieldArgs f{};
  f.dep_e = dep_buf(h, 0, 0);
  f.dep_i = dep_buf(h, 1, 0);
  f.pool_n = pool_levels(h);
  f.zero_a = dep_buf(h, 0, 1);
  f.zero_b = ion_step ? dep_buf(h, 1, 1) : nullptr;
  f.rho = h->rho;
  f.phi = h->phi;
  f.E = h->Ebuf[par];
  f.th_cp = h->th_cp;
  f.th_m = h->th_m;
  f.acc_ne = h->acc_ne;
  f.acc_ni = h->acc_ni;
  f.acc_w = h->acc_w;
  f.ctl = h->ctl;
  f.V = h->vtab[(size_t)(h->step % h->p.steps_per_cycle)];
  f.dx = h->dx;
  f.qfac32 = h->qfac32;
  f.nfac32 = h->nfac32;
  f.kpois = h->kpois;
  f.nx = h->nx;
  f.mode = field_mode_;
  f.measuring = h->measuring;
  f.parity = par;
  return f;
}

bool is_ion_step(const pic_handle* h, int64_t step) {
  return !(h->p.flags & PIC_FLAG_IMMOBILE_IONS) && (step % h->p.ion_subcycle == 0);
}

constexpr int kTailRareBlocks = 128;
// One-kernel steps use their small tiles up to this many particles per CU. us
// per step with small / large tiles, 512 cells, 256 CUs: 30 thousand of each
// species 16.4 / 21.0, 150 thousand 20.0 / 22.8, 400 thousand 26.6 / 27.2, 700
// thousand 34.5 / 33.6, 1 million 42.6 / 41.4, 2 million 74.6 / 66.9.
constexpr int64_t kStepSmall = 4096;
// What a tile costs more with every slot a candidate, in tiles without any.
// Workgroup times on the 64-discharge sweep: 13.4 us per tile at a candidate
// probability of 0.003, 15 at 0.03, 17 at 0.08, 22 at 0.24; the slowest workgroup
// decides, so a cost above the mean pays (40 steps: 48.9 ms at 3, 47.3 at 6, 50.1 at 1).
constexpr double kStepCandCost = 6.0;

// What one step of one discharge launches, in order:
//   [field(n)]  e_decide e_emit  [e_rare i_decide i_emit on ion steps]
//   then either the tail (queued slots of the last pass + field(n+1)) when
//   another step follows, or the last pass's rare kernel alone;
//   then a sort or repack of each species when due.
//
// Electron steps are pipelined when enabled and the schedule allows: the
// emit of step n then also decides step n+1 (k_emit_decide, which also runs
// step n's queued slots), so step n+1 has no decide pass and step n no tail.
// That needs the field of step n+1 before the emit of step n, so it applies
// to steps that are not the last of a call, not ion steps (the ions' deposit
// enters that field), not followed by a sort or repack (slots move) and not
// measuring:
//   [field(n)] [e_decide(n)] field_cand(n+1) e_emit_decide(n)
// A step whose electrons were decided that way (e_pushed) runs e_emit and
// the electron queued slots on the pushed state.
struct StepPlan {
  bool field_first;  // solve this step's field before the passes
  FieldArgs ff;
  bool measure;
  PartArgs ae;
  bool e_pushed;  // the previous step decided this step's electrons
  bool fuse;      // this step's electron emit decides the next step
  PartArgs ae_next;
  bool ion;
  PartArgs ai;
  int pend_sp;  // species of the last pass, whose queued slots run last
  bool tail;    // the next step's field is solved with those slots
  FieldArgs fn; // the next step's field (with the tail, or before the fused emit)
  int post;     // 0: nothing, 1: sort, 2: repack (both species)
  SortArgs sa[2];
};

void plan_post(pic_handle* h, int post, SortArgs* sa);

// What follows a step that ends at step index `step`: nothing (0), the stable
// sort by cell (1; the pool is rebuilt in the new slot order) or the pool
// rebuilt in slot order (2), which drops the entries of absorbed particles.
int post_of(const pic_params& p, int64_t step) {
  if (p.sort_interval > 0 && step % p.sort_interval == 0) return 1;
  if ((p.sort_interval == 0 || p.sort_interval > kRepackSteps) && step % kRepackSteps == 0) return 2;
  return 0;
}

// Plans the next step of h and advances the host-side schedule state past
// it (buffer parities, step index). field_ready: this step's field was
// solved by the previous step's tail; last: no step follows in this call.
StepPlan plan_step(pic_handle* h, bool field_ready, bool last, bool allow_fuse) {
  StepPlan q{};
  const pic_params& p = h->p;
  const int mode = field_mode(h);
  const int par = (int)(h->step & 1);
  q.ion = is_ion_step(h, h->step);
  q.field_first = !field_ready;
  if (q.field_first) q.ff = field_args(h, mode, q.ion);
  h->e_last = par;
  q.measure = h->measuring != 0;
  q.e_pushed = h->e_decided != 0;
  h->e_decided = 0;
  q.ae = particle_args(h, 0, par);
  h->cur[0] ^= 1;
  h->tsel[0] ^= 1;
  h->csel[0] ^= 1;
  q.pend_sp = 0;
  if (q.ion) {
    // the ions take this step's ionization ions with their velocities
    q.ai = particle_args(h, 1, par);
    h->cur[1] ^= 1;
    h->tsel[1] ^= 1;
    h->csel[1] ^= 1;
    h->dsel[1] = (h->dsel[1] + 1) % 3;
    q.pend_sp = 1;
  }
  h->dsel[0] = (h->dsel[0] + 1) % 3;
  h->dep_clean = 0;
  h->step += 1;
  q.post = post_of(p, h->step);
  q.fuse = allow_fuse && !last && !q.ion && q.post == 0 && !q.measure;
  q.tail = !last && !q.fuse;
  if (!last) q.fn = field_args(h, mode, is_ion_step(h, h->step));
  if (q.fuse) {
    // the next step's electron arguments, as its own plan will make them
    q.ae_next = particle_args(h, 0, (int)(h->step & 1));
    h->e_decided = 1;
    // with the next step's field, the candidacy bits of its electron slots
    // (their count is the sum of this step's output totals)
    FieldArgs& f = q.fn;
    f.cand = h->cand;
    f.cand_tcnt = q.ae.tcnt;
    f.cand_count = &h->ctl->n_e[par];
    f.cand_zero = q.ae_next.tcnt;
    f.cand_zero_n = h->max_tiles[0];
    f.cand_cap = h->p.capacity[0];
    f.cand_thr = q.ae_next.no_coll ? 0ull : q.ae_next.pcoll_thr;
    f.cand_step = q.ae_next.step;
    f.seed = h->p.seed;
    f.run = h->p.run;
  }
  plan_post(h, q.post, q.sa);
  return q;
}

// The sort or repack arguments of both species, and the schedule past them.
void plan_post(pic_handle* h, int post, SortArgs* sa) {
  for (int sp = 0; sp < 2 && post; ++sp) {
    sa[sp] = sort_args(h, sp, post == 1);
    if (post == 1) h->cur[sp] ^= 1;
    h->pcur[sp] ^= 1;
  }
}

int launch_post(pic_handle* h, int post, const SortArgs* sa, hipStream_t s) {
  if (post == 1 && h->timing == 0) {
    HIP_TRY(launch_sort(sa, 2, h->num_cu, s));
    return PIC_OK;
  }
  for (int sp = 0; sp < 2; ++sp) {
    if (post == 1) {
      const int ev = timer_begin(h);
      HIP_TRY(launch_sort(sa + sp, 1, h->num_cu, s));
      timer_end(h, PIC_TIMER_SORT, ev);
    } else if (post == 2) {
      HIP_TRY(launch_repack(sa[sp], s));
    }
  }
  return PIC_OK;
}

// One planned step on the handle's own stream, with the opt-in timers.
int launch_step(pic_handle* h, const StepPlan& q) {
  hipStream_t s = h->stream;
  if (q.field_first) {
    const int ev = timer_begin(h);
    HIP_TRY(launch_field(q.ff, s));
    timer_end(h, PIC_TIMER_FIELD, ev);
  }
  const int e_pass = timer_begin(h);
  if (!q.e_pushed) {
    const int ev = h->timing >= 2 ? timer_begin(h) : -1;
    HIP_TRY(launch_particle_kernel(0, 0, q.measure, q.ae, h->launch[0], s));
    timer_end(h, PIC_TIMER_E_DECIDE, ev);
  }
  if (q.fuse) {
    int ev = h->timing >= 2 ? timer_begin(h) : -1;
    HIP_TRY(launch_field_cand(q.fn, h->num_cu, s));
    timer_end(h, PIC_TIMER_FIELD, ev);
    ev = h->timing >= 2 ? timer_begin(h) : -1;
    HIP_TRY(launch_emit_decide(q.ae, q.ae_next, h->launch[0], s, q.e_pushed));
    timer_end(h, PIC_TIMER_E_EMIT, ev);
    timer_end(h, PIC_TIMER_ELECTRON, e_pass);
    return launch_post(h, q.post, q.sa, s);
  }
  const int pushed = q.e_pushed ? kLaunchPushed : 0;
  {
    const int ev = h->timing >= 2 ? timer_begin(h) : -1;
    HIP_TRY(launch_particle_kernel(1, 0, q.measure, q.ae, h->launch[0], s, pushed));
    timer_end(h, PIC_TIMER_E_EMIT, ev);
  }
  int pend_pass = e_pass;
  if (q.ion) {
    const int ev = h->timing >= 2 ? timer_begin(h) : -1;
    HIP_TRY(launch_particle_kernel(2, 0, q.measure, q.ae, h->launch[0], s, pushed));
    timer_end(h, PIC_TIMER_E_RARE, ev);
    timer_end(h, PIC_TIMER_ELECTRON, e_pass);
    const int i_pass = timer_begin(h);
    for (int k = 0; k < 2; ++k) {
      const int ev2 = h->timing >= 2 ? timer_begin(h) : -1;
      HIP_TRY(launch_particle_kernel(k, 1, false, q.ai, h->launch[1], s));
      timer_end(h, k == 0 ? PIC_TIMER_I_DECIDE : PIC_TIMER_I_EMIT, ev2);
    }
    pend_pass = i_pass;
  }
  const PartArgs& pend = q.pend_sp == 0 ? q.ae : q.ai;
  const int pend_pushed = q.pend_sp == 0 ? pushed : 0;
  const int ev = h->timing >= 2 ? timer_begin(h) : -1;
  if (q.tail)
    HIP_TRY(launch_tail(q.pend_sp, q.fn, pend, kTailRareBlocks, s, pend_pushed != 0));
  else
    HIP_TRY(launch_particle_kernel(2, q.pend_sp, q.measure, pend, h->launch[q.pend_sp], s,
                                   pend_pushed));
  timer_end(h, q.pend_sp == 0 ? PIC_TIMER_E_RARE : PIC_TIMER_I_RARE, ev);
  timer_end(h, q.pend_sp == 0 ? PIC_TIMER_ELECTRON : PIC_TIMER_ION, pend_pass);
  return launch_post(h, q.post, q.sa, s);
}

// n_steps steps with a kernel per pass.
int run_passes(pic_handle* h, int64_t n_steps) {
  bool field_ready = false;
  for (int64_t it = 0; it < n_steps; ++it) {
    const StepPlan q = plan_step(h, field_ready, it + 1 == n_steps, h->pipeline != 0);
    const int st = launch_step(h, q);
    if (st) return st;
    field_ready = q.tail || q.fuse;
    // keep the event backlog bounded
    if (h->ev_used.size() >= 4096) {
      const int c = timer_collect(h);
      if (c) return c;
    }
  }
  return PIC_OK;
}

// ---- one-kernel steps (k_step.hip) ----------------------------------------
// A run of steps n .. n + k is the launches
//   decide(n)  emit(n) + decide(n + 1)  ...  emit(n + k)
// where emit and decide of one launch cover both species (ions on their
// sub-cycled steps). A sort or repack moves slots, so the launch before one
// only emits and the launch after one only decides.

bool self_field(const pic_handle* h) {
  return field_mode(h) == FIELD_EXACT && h->nx <= kSelfMaxNx;
}

// A batch deals tiles to its workgroups by weight: collision candidates cost
// more than the streaming work of their tile as they become common.
int step_weight(const pic_handle* h, int sp) {
  const bool coll = (h->p.flags & PIC_FLAG_NO_COLL) == 0;
  return 16 + (coll ? (int)(16.0 * kStepCandCost * h->pcoll[sp]) : 0);
}

// Plans the launch that emits the current step (emit) and decides the step
// after it (decide; without emit, the current step), and advances the
// schedule past it. self_max: the largest grid whose workgroups solve the field
// themselves.
StepArgs plan_step_kernel(pic_handle* h, bool emit, bool decide, int self_max) {
  StepArgs a{};
  const int64_t ds = h->step + (emit ? 1 : 0);
  a.ctl = h->ctl;
  a.pool_in = h->ctl->pool_n[h->psel];
  a.pool_out = h->ctl->pool_n[h->psel ^ 1];
  for (int sp = 0; sp < 2; ++sp) {
    StepSpecies& s = a.sp[sp];
    s.emit = emit && (sp == 0 || is_ion_step(h, h->step));
    s.decide = decide && (sp == 0 || is_ion_step(h, ds));
    const bool move = s.emit || s.decide;
    const int in = h->cur[sp], out = move ? 1 - in : in;
    s.xin = h->part[sp][in][0];
    s.vxin = h->part[sp][in][1];
    s.idin = h->pid[sp][in];
    s.xout = h->part[sp][out][0];
    s.vxout = h->part[sp][out][1];
    s.idout = h->pid[sp][out];
    h->cur[sp] = out;
    s.pv = h->pool[sp][h->pcur[sp]];
    s.cin = h->codes[sp][h->csel[sp] ^ 1];
    s.cout = h->codes[sp][h->csel[sp]];
    s.tin = h->stc[sp][h->ssel[sp]];
    s.tout = h->stc[sp][(h->ssel[sp] + 1) % 3];
    s.tzero = h->stc[sp][(h->ssel[sp] + 2) % 3];
    s.ntz = (int)h->stc_n[sp];
    s.weight = step_weight(h, sp);
    if (s.decide) {
      h->csel[sp] ^= 1;
      h->ssel[sp] = (h->ssel[sp] + 1) % 3;
    }
    s.dep_in = dep_buf(h, sp, 0);
    s.dep_out = reinterpret_cast<unsigned long long*>(dep_buf(h, sp, 1));
    s.dep_zero = dep_buf(h, sp, 2);
    if (decide) h->dsel[sp] = (h->dsel[sp] + 1) % 3;
    s.cum = h->cum[sp];
    s.fedf = h->fedf[sp];
    s.cap = h->p.capacity[sp];
    s.pcap = h->pcap[sp];
    s.cand_thr = (h->p.flags & PIC_FLAG_NO_COLL) ? 0ull : candidacy_threshold(h->pcoll[sp]);
    s.acc = h->acc[sp];
    s.dts = h->dts[sp];
    s.p_wall = sp == 0 ? h->p.reflection : h->p.gamma_see;
    s.numax = h->numax[sp];
    s.inv_dv = h->inv_dv[sp];
    s.ek_s = 0.5 * h->mass[sp] / kQe;
    s.fedf_inv_de = (double)h->p.eepf_bins / h->fedf_emax[sp];
  }
  a.rho = h->rho;
  a.phi = h->phi;
  a.E = h->Ebuf[ds & 1];
  if (decide) h->e_last = (int)(ds & 1);
  a.acc_ne = h->acc_ne;
  a.acc_ni = h->acc_ni;
  a.acc_w = h->acc_w;
  a.acc_ew = h->acc_ew;
  a.eepf = h->eepf;
  a.V = h->vtab[(size_t)(ds % h->p.steps_per_cycle)];
  a.dx = h->dx;
  a.qfac32 = h->qfac32;
  a.nfac32 = h->nfac32;
  a.kpois = h->kpois;
  a.inv_dx = h->inv_dx;
  a.L = h->L;
  a.mr = h->mr_e;
  a.mm = h->mm_e;
  a.ek = h->ek_e;
  a.ve = h->ve_e;
  a.exc_thr = h->exc_thr;
  a.ion_thr = h->ion_thr;
  a.sig_g = h->sig_g;
  a.sig_se = h->sig_se;
  a.half = 0.5 * h->L;
  a.eepf_hw = h->p.eepf_halfwidth_m;
  a.inv_de = h->inv_de;
  a.nx = h->nx;
  a.ntab = h->ntab;
  a.nbins = h->p.eepf_bins;
  a.par = (int)(h->step & 1);
  a.self = self_field(h) && h->nx <= self_max ? 1 : 0;
  a.measuring = h->measuring;
  a.record = (h->p.flags & PIC_FLAG_RECORD) ? 1 : 0;
  a.model = ((h->p.flags & PIC_FLAG_ANISO_ELASTIC) ? kModelAniso : 0) |
            ((h->p.flags & PIC_FLAG_OPAL_SHARING) ? kModelOpal : 0);
  a.mstep = (uint32_t)h->step;
  a.dstep = (uint32_t)ds;
  a.seed = h->p.seed;
  a.run = h->p.run;
  if (emit) {
    h->psel ^= 1;
    h->step += 1;
  }
  return a;
}

// The field launch before a deciding step kernel that does not solve the
// field itself (the deposit buffers are the step kernel's to zero).
FieldArgs step_field_args(pic_handle* h, const StepArgs& a) {
  FieldArgs f{};
  f.dep_e = a.sp[0].dep_in;
  f.dep_i = a.sp[1].dep_in;
  f.rho = h->rho;
  f.phi = h->phi;
  f.E = a.E;
  f.th_cp = h->th_cp;
  f.th_m = h->th_m;
  f.acc_ne = h->acc_ne;
  f.acc_ni = h->acc_ni;
  f.acc_w = h->acc_w;
  f.ctl = h->ctl;
  f.V = a.V;
  f.dx = h->dx;
  f.qfac32 = h->qfac32;
  f.nfac32 = h->nfac32;
  f.kpois = h->kpois;
  f.nx = h->nx;
  f.mode = field_mode(h);
  f.measuring = h->measuring;
  f.parity = a.par;
  return f;
}

// The deposit buffers that the first deciding launch adds into have to be
// zero; the per-pass kernels leave them as they are.
int clean_deposits(pic_handle* h) {
  if (h->dep_clean) return PIC_OK;
  HIP_TRY(launch_clear2(dep_buf(h, 0, 1), dep_buf(h, 1, 1), h->nx, h->stream));
  h->dep_clean = 1;
  return PIC_OK;
}

// Slots per thread of the step kernel: small tiles until the particles fill
// the chip several times over.
int step_ppt(int64_t particles, int num_cu) {
  return particles <= (int64_t)num_cu * kStepSmall ? kStepPpt[1] : kStepPpt[0];
}

int64_t step_max_tiles(const pic_handle* h, int ppt) {
  const int64_t t = (int64_t)kBlock * ppt;
  return (h->p.capacity[0] + t - 1) / t + (h->p.capacity[1] + t - 1) / t + 1;
}

// The one-kernel steps' instance for the discharge as the host last saw it.
int step_plan_shape(pic_handle* h, StepShape* c) {
  const int ppt = step_ppt(h->hint[0] + h->hint[1], h->num_cu);
  *c = StepShape{ppt, h->measuring != 0,
                 (h->p.flags & (PIC_FLAG_ANISO_ELASTIC | PIC_FLAG_OPAL_SHARING)) != 0, 0, 0};
  int& fit = h->step_fit[ppt == kStepPpt[0]][c->measure];
  if (!fit) {
    HIP_TRY(step_fit(*c, false, h->nx, h->p.eepf_bins));
    fit = c->fit;
  }
  c->fit = fit;
  return PIC_OK;
}

// Whether one-kernel steps pay for a run of steps: by their instance's workgroups per CU (c.fit: registers hold it to
// three, a wide grid's LDS to two or one, while the per-pass kernels keep four),
// by how often the ions move (the passes skip resting ions and pipeline the
// electrons between) and by the steps of a run (a call, or the steps between
// two sorts: a run's first decisions and last emit are launches of their own).
//
// Up to how many million particles of both species a run of one step, of two
// and a long one takes them ([ions every step / every 2 to 5 / rarer or at
// rest], 0: always). From the ratio of one-kernel steps to passes, per million of
// each species, 512 to 4096 cells, ions every 1st / 3rd / 10th step, over a
// whole sort interval (long runs):
//   3 per CU                2 .60 / .76 / .80    4 .68 / .87 / .87   8 .66 / .91 / .92
//     measuring             2 .71 / .85 / .86    4 .80 / .92 / .83   8 .75 / .86 / .83
//   2 per CU, own field     2 .67 / .85 / .90    4 .74 / .99 / .99   6 .76 / 1.08 / 1.01
//     (in calls of 40 steps; 200 steps, growing, ions every 10th step: 9.6 million
//     in all 14.4 / 14.7 ms, 9.8 million 15.2 / 14.8)
//     field launch          2 .70 / .91 / .98    3 .74 / .97 / 1.02  4 .78 / 1.03 / 1.06
//     measuring             2 .78 / .97 / .98    4 .87 / 1.02 / .92  6 .89 / 1.01 / .94
//   1 per CU                0.4 .65 / .91 / .99  1 .81 / 1.03 / 1.12  4 1.08 / 1.31 / 1.39
//     measuring             0.15 .66 / .90 / .97 0.4 .86 / 1.08 / 1.07 2 1.12 / 1.31 / 1.23
// runs of one step:
//   3 per CU                1 .80 / .92 / .95    2 .93 / 1.0 / 1.04   4 1.13 / 1.08 / 1.07
//     measuring             0.4 .73 / .83 / .87  1 .94 / 1.02 / 1.05  4 1.13 / 1.05 / 1.02
//   2 per CU                1 .85 / .95 / 1.01   2 .98 / 1.06 / 1.09  4 1.23 / 1.16 / 1.16
//     measuring             0.4 .86 / .99 / 1.03 1 .94 / 1.05 / 1.08  4 1.24 / 1.13 / 1.08
//   1 per CU                0.4 .82 / 1.0 / 1.06 1 1.02 / 1.14 / 1.21 4 1.53 / 1.51 / 1.50
//     measuring             0.15 .82 / 1.0 / 1.08 0.4 1.06 / 1.13 / 1.15
struct StepLimit {
  float one, two, many;
};
constexpr StepLimit kStepLimit[3][2][3] = {
    // [workgroups per CU - 1][measuring][how often the ions move]
    {{{1.8f, 2.8f, 6.0f}, {0.8f, 1.7f, 1.7f}, {0.3f, 0.6f, 0.9f}},
     {{0.6f, 1.1f, 3.0f}, {0.3f, 0.5f, 0.6f}, {0.1f, 0.3f, 0.5f}}},
    {{{4.0f, 8.0f, 0.0f}, {2.6f, 5.4f, 8.0f}, {1.6f, 5.4f, 9.7f}},
     {{2.8f, 6.0f, 0.0f}, {1.0f, 3.4f, 5.0f}, {0.6f, 2.4f, 0.0f}}},
    {{{5.0f, 0.0f, 0.0f}, {3.8f, 8.0f, 0.0f}, {3.0f, 9.0f, 0.0f}},
     {{4.0f, 0.0f, 0.0f}, {1.8f, 7.0f, 0.0f}, {1.6f, 0.0f, 0.0f}}}};
// two per CU and the field in a launch of its own, ions not every step
constexpr StepLimit kStepLimitField[2] = {{2.0f, 4.0f, 7.0f}, {0.7f, 2.8f, 5.0f}};

bool step_kernel_pays(const pic_handle* h, const StepShape& c, int64_t n_steps) {
  const int fit = c.fit > 3 ? 3 : c.fit;
  const bool rest = (h->p.flags & PIC_FLAG_IMMOBILE_IONS) || h->p.ion_subcycle > 5;
  const int often = rest ? 2 : h->p.ion_subcycle > 1 ? 1 : 0;
  const bool own_launch = fit == 2 && !c.measure && often > 0 && !self_field(h);
  const StepLimit& l = own_launch ? kStepLimitField[often - 1] : kStepLimit[fit - 1][c.measure][often];
  int64_t run = n_steps;
  if (h->p.sort_interval > 0 && run > h->p.sort_interval) run = h->p.sort_interval;
  // (a field launch for the first decisions and none of the ions to save on:
  // 400 thousand of each species on 2400 cells 49 us against 44)
  if (run <= 1 && rest && !self_field(h)) return false;
  // from two steps on, the cost of a run's ends spreads over its steps
  const double many = l.many > 0.0f ? 1.0 / l.many : 0.0, two = l.two > 0.0f ? 1.0 / l.two : 0.0;
  const double inv = run <= 1 ? 1.0 / l.one : many + (two - many) / (double)(run - 1);
  return (double)(h->hint[0] + h->hint[1]) * 1e-6 * inv <= 1.0;
}

// Whether a call of n_steps takes one-kernel steps, and their instance.
int step_route(pic_handle* h, int64_t n_steps, StepShape* c, bool* one_kernel) {
  *one_kernel = false;
  if (!h->pipeline || h->timing != 0) return PIC_OK;
  const int st = step_plan_shape(h, c);
  if (!st) *one_kernel = step_kernel_pays(h, *c, n_steps);
  return st;
}

// Counts that the host does not wait for: asked for after this many steps
// without a reading call, so that the schedule of a discharge that grows or
// shrinks meanwhile follows it (a launch of about 3 us). Loaded with 400 thousand
// and grown to 4 million of each species unread, a discharge would keep the
// small tiles: 2048 cells, ions every 10th step 74 us per step against 66, 4096
// cells measuring 362 against 233.
constexpr int64_t kLookSteps = 256;

int ask_counts(pic_handle* h) {
  if (h->unseen < kLookSteps) return PIC_OK;
  h->unseen = 0;
  HIP_TRY(launch_counts(h->ctl, (int)(h->step & 1), h->seen, h->stream));
  return PIC_OK;
}

// What has arrived of them.
void take_counts(pic_handle* h) {
  for (int sp = 0; sp < 2; ++sp) {
    const int64_t n = static_cast<volatile int64_t*>(h->seen)[sp];
    if (n >= 0) saw_count(h, sp, n);
  }
}

// Up to n_steps one-kernel steps, *done of them: to the first sort or repack
// after which the counts are looked at again.
int run_step_kernels(pic_handle* h, int64_t n_steps, StepShape c, int64_t* done) {
  step_grid(c, h->num_cu, h->step_wg, step_max_tiles(h, c.ppt));
  const int st = clean_deposits(h);
  if (st) return st;
  auto launch = [&](bool emit, bool decide) -> int {
    const StepArgs a = plan_step_kernel(h, emit, decide, kSelfMaxNx);
    if (decide && !a.self) HIP_TRY(launch_field(step_field_args(h, a), h->stream));
    HIP_TRY(launch_step_kernel(a, c, h->stream));
    return PIC_OK;
  };
  bool decided = false;
  for (*done = 0; *done < n_steps;) {
    int e = decided ? PIC_OK : launch(false, true);
    if (e) return e;
    const int post = post_of(h->p, h->step + 1);
    decided = *done + 1 < n_steps && post == 0;
    e = launch(true, decided);
    if (e) return e;
    if (post) {
      SortArgs sa[2];
      plan_post(h, post, sa);
      e = launch_post(h, post, sa, h->stream);
      if (e) return e;
    }
    *done += 1;
    h->unseen += 1;
    if (post && h->unseen >= kLookSteps) break;
  }
  return PIC_OK;
}

// Batched stepping: the argument blocks of every discharge's launches go to
// device memory (one upload per chunk of steps, double buffered through
// pinned host memory) and each launch covers all discharges.
constexpr size_t kBatchUploadBytes = (size_t)8 << 20;  // per chunk buffer
constexpr size_t kBatchArrayAlign = 64;

// most workgroups of a batch launch
int batch_max_wgs(int num_cu) { return 8 * num_cu + kMaxBatch; }

// Deals the workgroups of a batch to its discharges: one each, then always
// one more to the discharge with the most work per workgroup (its particles
// as the host last saw them, weighted as the kernel weighs its tiles).
void deal_workgroups(const std::vector<pic_handle*>& hs, int grid, StepWg* out) {
  const int n = (int)hs.size();
  std::vector<double> work(n);
  std::vector<int> g(n, 1);
  typedef std::pair<double, int> Share;
  std::priority_queue<Share> heap;
  for (int i = 0; i < n; ++i) {
    const pic_handle* h = hs[i];
    const bool mobile = (h->p.flags & PIC_FLAG_IMMOBILE_IONS) == 0;
    work[i] = 1.0 + (double)h->hint[0] * step_weight(h, 0) +
              (mobile ? (double)h->hint[1] * step_weight(h, 1) / h->p.ion_subcycle : 0.0);
    heap.push(Share(work[i], i));
  }
  for (int left = grid - n; left > 0; --left) {
    const int i = heap.top().second;
    heap.pop();
    g[i] += 1;
    heap.push(Share(work[i] / g[i], i));
  }
  int b = 0;
  for (int i = 0; i < n; ++i)
    for (int k = 0; k < g[i]; ++k) out[b++] = StepWg{i, k, g[i], 0};
}

size_t batch_align(size_t v) {
  return (v + kBatchArrayAlign - 1) / kBatchArrayAlign * kBatchArrayAlign;
}

// Upload bytes of a step on the route that takes more.
size_t batch_step_bytes(int n) {
  // one kernel: the deciding launch of the discharges that start or follow a
  // sort, the launch that emits, the field launches before both. Passes: the
  // fields before and after, the electron decide, the electron queued slots of
  // ion steps, the ions, the queued slots otherwise. Both: the sorts of both
  // species
  const size_t f = 2 * batch_align((size_t)n * sizeof(FieldArgs));
  const size_t one = 2 * batch_align((size_t)n * sizeof(StepArgs));
  const size_t pass = 4 * batch_align((size_t)n * sizeof(PartArgs));
  return f + (one > pass ? one : pass) + 2 * batch_align((size_t)n * sizeof(SortArgs));
}

int batch_chunk_steps(int n) {
  const size_t per = batch_step_bytes(n);
  size_t c = kBatchUploadBytes / per;
  if (c < 1) c = 1;
  if (c > 64) c = 64;
  return (int)c;
}

// one of a batch's two upload buffers
size_t batch_half_bytes(int n, int num_cu) {
  const size_t wg = batch_align((size_t)batch_max_wgs(num_cu) * sizeof(StepWg));
  const size_t b = (size_t)batch_chunk_steps(n) * batch_step_bytes(n) + wg +
                   batch_align((size_t)n * sizeof(BatchCount));
  return (b + kAlign - 1) / kAlign * kAlign;
}

int check_batch_handles(pic_handle* const* hs, int n) {
  if (!hs || n < 1 || n > kMaxBatch) return PIC_EINVAL;
  for (int i = 0; i < n; ++i) {
    if (!hs[i]) return PIC_EINVAL;
    if (hs[i]->stream != hs[0]->stream || hs[i]->device != hs[0]->device) return PIC_EINVAL;
    for (int k = 0; k < i; ++k)
      if (hs[k] == hs[i]) return PIC_EINVAL;
  }
  return PIC_OK;
}

// The particle counts come back to the host by themselves once per chunk's
// worth of steps, and the schedule follows them (an older value only deals the
// workgroups less evenly). What the host saw or set since (it waited for the
// stream then) comes first.
void take_batch_counts(pic_batch* b) {
  for (size_t i = 0; i < b->hs.size(); ++i) {
    pic_handle* h = b->hs[i];
    if (h->hint_new) {
      b->counts[2 * i] = b->counts[2 * i + 1] = -1;
      h->hint_new = 0;
    }
    for (int sp = 0; sp < 2; ++sp) {
      const int64_t v = static_cast<volatile int64_t*>(b->counts)[2 * i + sp];
      if (v >= 0) {
        h->hint[sp] = v;
        h->seen[sp] = -1;
      }
    }
  }
}

// The batch's one-kernel instance and grid as the host last saw its discharges.
int batch_plan_shape(pic_batch* b, StepShape* c) {
  int64_t particles = 0, tiles = 0;
  bool measure = false;
  for (pic_handle* h : b->hs) {
    particles += h->hint[0] + h->hint[1];
    measure = measure || h->measuring;
  }
  const int ppt = step_ppt(particles, b->num_cu);
  for (pic_handle* h : b->hs) tiles += step_max_tiles(h, ppt);
  *c = StepShape{ppt, measure, b->variants, 0, 0};
  int& fit = b->step_fit[ppt == kStepPpt[0]][measure];
  if (!fit) {
    HIP_TRY(step_fit(*c, true, b->nx_max, b->nbins_max));
    fit = c->fit;
  }
  c->fit = fit;
  step_grid(*c, b->num_cu, 8, tiles);
  const int n = (int)b->hs.size();
  if (c->grid < n) c->grid = n;
  return PIC_OK;
}

// Up to how many million particles in all a batch's runs of one step and long
// ones take one kernel per step (kStepLimit's classes; the bound of a run of r
// steps goes from the one to the other with 1/r^2, which holds at 2 and 4 steps).
// A batch saves one set of launches for all its discharges either way, so the
// passes are ahead from smaller totals than for one discharge. Ratio of
// one-kernel steps to passes, ions every 1st / 3rd / 10th step, totals in
// millions (discharges x particles):
//   in calls of 100 steps    0.5 (100x5k)     3.2 (64x50k)     4 (4x1M)          8 (2x4M)
//     1200 cells, 3 per CU   .35 .45 .50      .55 .70 .65      .67 .85 .78       .69 .87 .80
//       measuring            .38 .50 .58      .63 .82 .76      .73 .92 .85       .71 .85 .77
//     2048 cells, 2 per CU   .37 .49 .54      .59 .75 .73      .71 .91 .86       .72 .95 .90
//       measuring            .47 .61 .65      .72 .93 .88      .82 1.04 .95      .86 1.01 .93
//     4096 cells, 1 per CU   .45 .61 .66      .74 .95 .93      .93 1.21 1.11     .97 1.24 1.14
//     2400, measuring        .52 .68 .75      .97 1.23 1.14    1.18 1.47 1.32    1.25 1.46 1.26
//   in calls of one step
//     1200 cells             .68 .85 .94      1.0 1.08 1.11    1.14 1.19 1.21    1.19 1.26 1.31
//       measuring            .67 .81 .91      1.0 1.04 1.04    1.13 1.17 1.21    1.15 1.13 1.12
//     2048 cells             .68 .86 .93      .97 1.09 1.15    1.10 1.18 1.24    1.18 1.26 1.31
//       measuring            .67 .80 .86      1.04 1.06 1.09   1.21 1.23 1.28    1.23 1.24 1.24
//     4096 cells             .67 .83 .94      1.06 1.14 1.21   1.34 1.36 1.38    1.40 1.48 1.55
//     2400, measuring        .67 .81 .87      1.28 1.30 1.28   1.52 1.53 1.51    1.64 1.58 1.53
struct BatchLimit {
  float one, many;  // many 0: no bound
};
constexpr BatchLimit kBatchLimit[3][2][3] = {
    // [workgroups per CU - 1][measuring][how often the ions move]
    {{{1.4f, 9.0f}, {0.8f, 3.6f}, {0.55f, 3.6f}}, {{1.2f, 3.3f}, {0.6f, 0.9f}, {0.6f, 0.75f}}},
    {{{3.3f, 0.0f}, {1.0f, 10.0f}, {0.7f, 10.0f}}, {{2.4f, 12.0f}, {0.9f, 3.6f}, {0.6f, 9.0f}}},
    {{{3.2f, 0.0f}, {1.2f, 0.0f}, {0.8f, 0.0f}}, {{3.3f, 0.0f}, {1.6f, 0.0f}, {0.9f, 0.0f}}}};

// Whether a batch's run of steps takes one kernel per step (step_kernel_pays
// for a discharge alone).
bool batch_kernel_pays(const pic_batch* b, const StepShape& c, int64_t n_steps) {
  double all = 0.0, ions = 0.0, moved = 0.0;
  int64_t run = n_steps;
  for (const pic_handle* h : b->hs) {
    all += (double)(h->hint[0] + h->hint[1]);
    ions += (double)h->hint[1];
    if (!(h->p.flags & PIC_FLAG_IMMOBILE_IONS)) moved += (double)h->hint[1] / h->p.ion_subcycle;
    if (h->p.sort_interval > 0 && run > h->p.sort_interval) run = h->p.sort_interval;
  }
  const int fit = c.fit > 3 ? 3 : c.fit;
  const int often = moved > 0.6 * ions ? 0 : moved > 0.18 * ions ? 1 : 2;
  const BatchLimit& l = kBatchLimit[fit - 1][c.measure][often];
  const double many = l.many > 0.0f ? 1.0 / l.many : 0.0;
  const double inv = many + (1.0 / l.one - many) / ((double)run * (double)run);
  return all * 1e-6 * inv <= 1.0;
}

// The upload buffer of a chunk of steps.
struct BatchUpload {
  unsigned char* H;
  unsigned char* D;
  size_t off;
  int slot;
  size_t take(size_t bytes) {
    const size_t o = off;
    off += batch_align(bytes);
    return o;
  }
};

int batch_open(pic_batch* b, BatchUpload* u) {
  *u = BatchUpload{b->host[b->slot], b->dev[b->slot], 0, b->slot};
  b->slot ^= 1;
  // the last upload from this host buffer has been read
  HIP_TRY(hipEventSynchronize(b->copied[u->slot]));
  return PIC_OK;
}

// Uploads a planned chunk of m steps; *counts: what launch_batch_counts takes
// after it, null while the counts are recent (their launch is 3 to 4 us, which
// a call of one step would pay each time).
int batch_send(pic_batch* b, BatchUpload* u, int m, const BatchCount** counts) {
  *counts = nullptr;
  b->unseen += m;
  if (b->unseen >= b->chunk) {
    b->unseen = 0;
    const size_t n = b->hs.size(), o = u->take(n * sizeof(BatchCount));
    BatchCount* c = reinterpret_cast<BatchCount*>(u->H + o);
    for (size_t i = 0; i < n; ++i) c[i] = BatchCount{b->hs[i]->ctl, b->hs[i]->step & 1};
    *counts = reinterpret_cast<const BatchCount*>(u->D + o);
  }
  HIP_TRY(hipMemcpyAsync(u->D, u->H, u->off, hipMemcpyHostToDevice, b->stream));
  HIP_TRY(hipEventRecord(b->copied[u->slot], b->stream));
  return PIC_OK;
}

// What follows a batch's step: the sorts due (arguments in the upload) and the
// repacks, launched one by one.
struct BatchPost {
  const SortArgs* so[2];
  SortArgs* host[2];
  int n;
  SortShape shape;
};

BatchPost batch_post(BatchUpload* u, int n) {
  BatchPost q{};
  for (int sp = 0; sp < 2; ++sp) {
    const size_t o = u->take((size_t)n * sizeof(SortArgs));
    q.so[sp] = reinterpret_cast<const SortArgs*>(u->D + o);
    q.host[sp] = reinterpret_cast<SortArgs*>(u->H + o);
  }
  return q;
}

struct BatchRepack {
  int step;
  int discharge;
  SortArgs sa[2];
};

void batch_add_post(BatchPost* q, std::vector<BatchRepack>* repacks, int step, int discharge,
                    int post, const SortArgs* sa) {
  if (post == 1) {
    for (int sp = 0; sp < 2; ++sp) q->host[sp][q->n] = sa[sp];
    q->n += 1;
  } else if (post) {
    repacks->push_back(BatchRepack{step, discharge, {sa[0], sa[1]}});
  }
}

// after a step's discharges
void batch_end_post(const pic_batch* b, BatchPost* q) {
  if (q->n) q->shape = sort_chunks(q->host[0], q->host[1], q->n, b->nx_max, b->num_cu);
}

int batch_launch_post(pic_batch* b, const BatchPost& q, const std::vector<BatchRepack>& repacks,
                      size_t* next, int step) {
  if (q.n) HIP_TRY(launch_batch_sort(q.so[0], q.so[1], q.n, q.shape, b->nx_max, b->stream));
  for (; *next < repacks.size() && repacks[*next].step == step; ++*next) {
    const BatchRepack& r = repacks[*next];
    const int st = launch_post(b->hs[r.discharge], 2, r.sa, b->stream);
    if (st) return st;
  }
  return PIC_OK;
}

// n_steps steps of every discharge, one kernel each. The discharges' fields are
// solved by a launch before it from 1026 points on (of many discharges at once
// it costs less than what every workgroup spends on 2049 points).
int batch_step_kernels(pic_batch* b, int64_t n_steps, const StepShape& c) {
  const int n = (int)b->hs.size();
  for (pic_handle* h : b->hs) {
    const int st = clean_deposits(h);
    if (st) return st;
  }
  std::vector<StepWg> wgs(c.grid);
  // one step's launches: device addresses of its argument arrays and counts
  struct StepLaunch {
    const FieldArgs* f[2];  // [0] the deciding launch, [1] the emitting one
    const StepArgs* a[2];
    int nf[2], na[2];
    BatchPost post;
  };
  std::vector<char> decided(n, 0);
  std::vector<StepLaunch> steps;
  std::vector<BatchRepack> repacks;
  for (int64_t done = 0; done < n_steps;) {
    const int m = (int)((n_steps - done < b->chunk) ? n_steps - done : b->chunk);
    BatchUpload u;
    int st = batch_open(b, &u);
    if (st) return st;
    steps.clear();
    repacks.clear();
    take_batch_counts(b);
    deal_workgroups(b->hs, c.grid, wgs.data());
    std::memcpy(u.H + u.take(c.grid * sizeof(StepWg)), wgs.data(), c.grid * sizeof(StepWg));
    for (int k = 0; k < m; ++k) {
      const bool last = done + k + 1 == n_steps;
      StepLaunch L{};
      // a deciding launch only if some discharge needs it; the others sit it
      // out (their argument blocks say so)
      bool any = false;
      for (int i = 0; i < n; ++i) any = any || !decided[i];
      const int nd = any ? n : 0;
      const size_t o_a[2] = {u.take(nd * sizeof(StepArgs)), u.take(n * sizeof(StepArgs))};
      const size_t o_f[2] = {u.take(nd * sizeof(FieldArgs)), u.take(n * sizeof(FieldArgs))};
      L.post = batch_post(&u, n);
      for (int q = 0; q < 2; ++q) {
        L.a[q] = reinterpret_cast<const StepArgs*>(u.D + o_a[q]);
        L.f[q] = reinterpret_cast<const FieldArgs*>(u.D + o_f[q]);
      }
      auto add = [&](int q, pic_handle* h, bool emit, bool decide) {
        const StepArgs a = plan_step_kernel(h, emit, decide, kSelfSmallNx);
        reinterpret_cast<StepArgs*>(u.H + o_a[q])[L.na[q]++] = a;
        if (decide && !a.self)
          reinterpret_cast<FieldArgs*>(u.H + o_f[q])[L.nf[q]++] = step_field_args(h, a);
      };
      for (int i = 0; i < n; ++i) {
        pic_handle* h = b->hs[i];
        if (!decided[i])
          add(0, h, false, true);
        else if (any)
          reinterpret_cast<StepArgs*>(u.H + o_a[0])[L.na[0]++] = StepArgs{};
        const int post = post_of(h->p, h->step + 1);
        decided[i] = !last && post == 0;
        add(1, h, true, decided[i] != 0);
        if (post) {
          SortArgs sa[2];
          plan_post(h, post, sa);
          batch_add_post(&L.post, &repacks, k, i, post, sa);
        }
      }
      batch_end_post(b, &L.post);
      steps.push_back(L);
    }
    const BatchCount* counts;
    st = batch_send(b, &u, m, &counts);
    if (st) return st;
    size_t next = 0;
    for (int k = 0; k < m; ++k) {
      const StepLaunch& L = steps[k];
      for (int q = 0; q < 2; ++q) {
        if (L.nf[q]) HIP_TRY(launch_batch_field(L.f[q], L.nf[q], b->stream));
        if (L.na[q])
          HIP_TRY(launch_step_batch(L.a[q], reinterpret_cast<const StepWg*>(u.D), c, b->nx_max,
                                    b->nbins_max, b->stream));
      }
      st = batch_launch_post(b, L.post, repacks, &next, k);
      if (st) return st;
    }
    if (counts) HIP_TRY(launch_batch_counts(counts, n, b->counts, b->stream));
    done += m;
  }
  return PIC_OK;
}

// n_steps steps of every discharge with a launch per pass for all of them.
int batch_passes(pic_batch* b, int64_t n_steps) {
  const int n = (int)b->hs.size();
  hipStream_t s = b->stream;
  const BatchLaunch& c = b->passes;
  // one step's launches: device addresses of its argument arrays and counts
  struct PassLaunch {
    const FieldArgs* ff;  // fields before the passes (a run's first step)
    const FieldArgs* fn;  // the next step's fields, with the tail
    const PartArgs* ed;   // measuring discharges first
    const PartArgs* er;   // electrons of ion steps, whose queued slots come before
    const PartArgs* ia;   // the ions
    const PartArgs* t0;   // electrons of the other steps
    int nff, nem, nion, nt0;
    bool tail;
    BatchPost post;
  };
  std::vector<StepPlan> plans(n);
  std::vector<PassLaunch> steps;
  std::vector<BatchRepack> repacks;
  bool field_ready = false;
  for (int64_t done = 0; done < n_steps;) {
    const int m = (int)((n_steps - done < b->chunk) ? n_steps - done : b->chunk);
    BatchUpload u;
    int st = batch_open(b, &u);
    if (st) return st;
    steps.clear();
    repacks.clear();
    for (int k = 0; k < m; ++k) {
      const bool last = done + k + 1 == n_steps;
      for (int i = 0; i < n; ++i) plans[i] = plan_step(b->hs[i], field_ready, last, false);
      field_ready = !last;
      PassLaunch L{};
      L.tail = !last;
      const size_t o_f[2] = {u.take(n * sizeof(FieldArgs)), u.take(n * sizeof(FieldArgs))};
      size_t o_p[4];
      for (size_t& o : o_p) o = u.take(n * sizeof(PartArgs));
      L.post = batch_post(&u, n);
      FieldArgs* ff = reinterpret_cast<FieldArgs*>(u.H + o_f[0]);
      FieldArgs* fn = reinterpret_cast<FieldArgs*>(u.H + o_f[1]);
      PartArgs* pa[4];
      for (int q = 0; q < 4; ++q) pa[q] = reinterpret_cast<PartArgs*>(u.H + o_p[q]);
      int ne = 0;
      for (int pass = 0; pass < 2; ++pass)
        for (int i = 0; i < n; ++i)
          if (plans[i].measure == (pass == 0)) {
            pa[0][ne++] = plans[i].ae;
            if (pass == 0) L.nem += 1;
          }
      for (int i = 0; i < n; ++i) {
        const StepPlan& q = plans[i];
        if (q.field_first) ff[L.nff++] = q.ff;
        if (L.tail) fn[i] = q.fn;
        if (q.ion) {
          pa[1][L.nion] = q.ae;
          pa[2][L.nion++] = q.ai;
        } else {
          pa[3][L.nt0++] = q.ae;
        }
        batch_add_post(&L.post, &repacks, k, i, q.post, q.sa);
      }
      L.ff = reinterpret_cast<const FieldArgs*>(u.D + o_f[0]);
      L.fn = reinterpret_cast<const FieldArgs*>(u.D + o_f[1]);
      const PartArgs** to[4] = {&L.ed, &L.er, &L.ia, &L.t0};
      for (int q = 0; q < 4; ++q) *to[q] = reinterpret_cast<const PartArgs*>(u.D + o_p[q]);
      batch_end_post(b, &L.post);
      steps.push_back(L);
    }
    const BatchCount* counts;
    st = batch_send(b, &u, m, &counts);
    if (st) return st;
    size_t next = 0;
    for (int k = 0; k < m; ++k) {
      const PassLaunch& L = steps[k];
      auto pass = [&](int kernel, int sp, bool measure, const PartArgs* a, int na) {
        return na ? launch_batch_pass(kernel, sp, measure, a, na, c, s, b->variants) : hipSuccess;
      };
      if (L.nff) HIP_TRY(launch_batch_field(L.ff, L.nff, s));
      HIP_TRY(pass(0, 0, true, L.ed, L.nem));
      HIP_TRY(pass(0, 0, false, L.ed + L.nem, n - L.nem));
      HIP_TRY(pass(1, 0, false, L.ed, n));
      HIP_TRY(pass(2, 0, false, L.er, L.nion));
      HIP_TRY(pass(0, 1, false, L.ia, L.nion));
      HIP_TRY(pass(1, 1, false, L.ia, L.nion));
      // the queued slots of the last pass, with the next fields if a step follows
      if (L.tail && L.nion)
        HIP_TRY(launch_batch_tail(1, L.fn, n, L.ia, L.nion, kTailRareBlocks, s, b->variants));
      else if (L.tail)
        HIP_TRY(launch_batch_tail(0, L.fn, n, L.t0, L.nt0, kTailRareBlocks, s, b->variants));
      else
        HIP_TRY(pass(2, 1, false, L.ia, L.nion));
      if (!L.tail || L.nion) HIP_TRY(pass(2, 0, false, L.t0, L.nt0));
      st = batch_launch_post(b, L.post, repacks, &next, k);
      if (st) return st;
    }
    if (counts) HIP_TRY(launch_batch_counts(counts, n, b->counts, s));
    done += m;
  }
  return PIC_OK;
}

// Replaces the particles of one species: fill(args) enqueues what writes the
// n particles to the active slot buffers and pool, their pool indices and
// deposit, from the argument block prepared here. Synchronises.
template <typename Fill>
int replace_state(pic_handle* h, int species, int64_t n, int64_t step, Fill fill) {
  h->e_decided = 0;
  InstallArgs a{};
  a.ctl = h->ctl;
  a.pool_n = &pool_levels(h)[species];
  a.dep = dep_buf(h, species, 0);
  a.x = h->part[species][h->cur[species]][0];
  a.vx = h->part[species][h->cur[species]][1];
  a.pv = h->pool[species][h->pcur[species]];
  a.id = h->pid[species][h->cur[species]];
  a.n = n;
  a.inv_dx = h->inv_dx;
  a.nx = h->nx;
  a.species = species;
  a.old_par = (int)(h->step & 1);
  a.par = (int)(step & 1);
  HIP_TRY(launch_install_begin(a, h->stream));
  h->step = step;
  saw_count(h, species, n);
  if (n > 0) {
    const int st = fill(a);
    if (st) return st;
  }
  HIP_TRY(hipStreamSynchronize(h->stream));
  h->seen[species] = -1;
  return PIC_OK;
}

}  // namespace

extern "C" {

const char* pic_strerror(int s) {
  switch (s) {
    case PIC_OK: return "ok";
    case PIC_EINVAL: return "invalid argument or parameter set";
    case PIC_EHIP: return "HIP runtime error (no GPU, or a launch failed)";
    case PIC_ECAPACITY: return "a species outgrew its capacity";
    case PIC_EUNSTABLE: return "non-finite position, velocity or field";
    case PIC_ETABLE: return "reserved";
    case PIC_ESTATE: return "call not valid in the current state";
    default: return "unknown status";
  }
}

int pic_workspace_bytes(const pic_params* p, const pic_xsec* xs, uint64_t* bytes) {
  if (!bytes) return PIC_EINVAL;
  const int v = validate(p, xs);
  if (v) return v;
  *bytes = make_layout(p, xs).total;
  return PIC_OK;
}

int pic_init(const pic_params* p, const pic_xsec* xs, void* workspace, uint64_t workspace_bytes,
             void* stream, pic_handle** out) {
  if (!out) return PIC_EINVAL;
  *out = nullptr;
  int v = validate(p, xs);
  if (v) return v;
  const Layout L = make_layout(p, xs);
  if (!workspace || workspace_bytes < L.total || ((uintptr_t)workspace % kAlign) != 0)
    return PIC_EINVAL;
  pic_handle* h = new (std::nothrow) pic_handle();
  if (!h) return PIC_EINVAL;
  h->p = *p;
  h->stream = (hipStream_t)stream;
  if (hipGetDevice(&h->device) != hipSuccess ||
      hipDeviceGetAttribute(&h->num_cu, hipDeviceAttributeMultiprocessorCount, h->device) !=
          hipSuccess) {
    delete h;
    return PIC_EHIP;
  }

  // ---- derived constants (Sec. 2): the operation order is part of the
  // method's definition, so every side computes them the same way
  h->nx = p->n_cells + 1;
  h->L = p->gap_m;
  h->dx = p->gap_m / (double)p->n_cells;
  h->inv_dx = 1.0 / h->dx;
  h->dt = 1.0 / (p->rf_freq_hz * (double)p->steps_per_cycle);
  h->ng = p->pressure_pa / (kKb * p->gas_temp_k);
  h->mass[0] = kMe;
  h->mass[1] = 39.948 * kAmu;
  h->dts[0] = h->dt;
  h->dts[1] = (double)p->ion_subcycle * h->dt;
  h->acc[0] = (-kQe / h->mass[0]) * h->dts[0];
  h->acc[1] = (kQe / h->mass[1]) * h->dts[1];
  h->nfac32 = p->weight / (p->area_m2 * h->dx) * kInvTwo32;
  h->qfac32 = kQe * h->nfac32;
  h->kpois = h->dx * h->dx * h->qfac32 / kEps0;
  h->inv_dv[0] = 1.0 / xs->dv_e;
  h->inv_dv[1] = 1.0 / xs->dv_i;
  h->ntab = xs->n;
  h->exc_thr = xs->exc_threshold_ev;
  h->ion_thr = xs->ion_threshold_ev;
  h->ek_e = 0.5 * kMe / kQe;
  h->ve_e = 2.0 * kQe / kMe;
  h->mr_e = kMe / (kMe + h->mass[1]);
  h->mm_e = h->mass[1] / (kMe + h->mass[1]);
  h->sig_g = std::sqrt(kKb * p->gas_temp_k / h->mass[1]);
  h->sig_se = std::sqrt(p->see_temp_ev * kQe / kMe);
  h->eepf_de = p->eepf_emax_ev / (double)p->eepf_bins;
  h->inv_de = (double)p->eepf_bins / p->eepf_emax_ev;

  // cumulative collision frequencies nu_k(v) = n_g sigma_k(v) v on the table
  // speeds, and nu_max over the table (Sec. 3.5)
  std::vector<double> cum[2];
  const double* sig[2][3] = {{xs->sigma_e[0], xs->sigma_e[1], xs->sigma_e[2]},
                             {xs->sigma_i[0], xs->sigma_i[1], nullptr}};
  const int nproc[2] = {3, 2};
  const double dv[2] = {xs->dv_e, xs->dv_i};
  for (int s = 0; s < 2; ++s) {
    cum[s].assign((size_t)nproc[s] * xs->n, 0.0);
    h->numax[s] = 0.0;
    for (int i = 0; i < xs->n; ++i) {
      const double vel = (double)i * dv[s];
      double run = 0.0;
      for (int k = 0; k < nproc[s]; ++k) {
        const double nu = h->ng * sig[s][k][i] * vel;
        run = (k == 0) ? nu : run + nu;
        cum[s][(size_t)i * nproc[s] + k] = run;
      }
      if (run > h->numax[s]) h->numax[s] = run;
    }
    h->pcoll[s] = 1.0 - std::exp(-h->numax[s] * h->dts[s]);
  }
  h->vtab.resize(p->steps_per_cycle);
  for (int m = 0; m < p->steps_per_cycle; ++m)
    h->vtab[m] = p->rf_voltage_v * std::cos(kTwoPi * (double)m / (double)p->steps_per_cycle);
  // Thomas recurrence coefficients of the constant [1, -2, 1] matrix
  std::vector<double> th_cp(h->nx, 0.0), th_m(h->nx, 0.0);
  {
    const int n = h->nx - 2;
    th_cp[0] = 1.0 / -2.0;
    th_m[0] = -2.0;
    for (int i = 1; i < n; ++i) {
      const double m = -2.0 - 1.0 * th_cp[i - 1];
      th_m[i] = m;
      th_cp[i] = 1.0 / m;
    }
  }

  // ---- workspace
  char* w = static_cast<char*>(workspace);
  h->ctl = reinterpret_cast<DevCtl*>(w + L.ctl);
  for (int s = 0; s < 2; ++s) {
    for (int b = 0; b < 2; ++b) {
      for (int q = 0; q < 2; ++q)
        h->part[s][b][q] = reinterpret_cast<double*>(w + L.part[s][b][q]);
      h->pool[s][b] = reinterpret_cast<double2*>(w + L.pool[s][b]);
      h->pid[s][b] = reinterpret_cast<uint32_t*>(w + L.pid[s][b]);
    }
    h->pcap[s] = pool_capacity(p->capacity[s]);
    for (int b = 0; b < 2; ++b) h->codes[s][b] = reinterpret_cast<uint8_t*>(w + L.codes[s][b]);
    h->csel[s] = 0;
    for (int b = 0; b < 2; ++b) h->tcnt[s][b] = reinterpret_cast<uint64_t*>(w + L.tcnt[s][b]);
    h->tsel[s] = 0;
    h->rq[s] = reinterpret_cast<uint4*>(w + L.rq[s]);
    h->max_tiles[s] = L.max_tiles[s];
    h->cum[s] = reinterpret_cast<double*>(w + L.cum[s]);
  }
  for (int s = 0; s < 2; ++s) {
    for (int b = 0; b < 3; ++b) {
      h->dep[s][b] = reinterpret_cast<int64_t*>(w + L.dep[s][b]);
      h->stc[s][b] = reinterpret_cast<uint32_t*>(w + L.stc[s][b]);
    }
    h->dsel[s] = h->ssel[s] = 0;
    h->stc_n[s] = L.stc_n[s];
    h->hint[s] = 0;
  }
  h->dep_clean = 1;
  h->psel = 0;
  h->step_wg = 0;
  for (int k = 0; k < 4; ++k) h->step_fit[k / 2][k % 2] = 0;
  h->rho = reinterpret_cast<double*>(w + L.rho);
  h->phi = reinterpret_cast<double*>(w + L.phi);
  for (int b = 0; b < 2; ++b) h->Ebuf[b] = reinterpret_cast<double*>(w + L.E[b]);
  h->e_last = 0;
  h->th_cp = reinterpret_cast<double*>(w + L.th_cp);
  h->th_m = reinterpret_cast<double*>(w + L.th_m);
  h->acc_ne = reinterpret_cast<double*>(w + L.acc_ne);
  h->acc_ni = reinterpret_cast<double*>(w + L.acc_ni);
  h->acc_w = reinterpret_cast<double*>(w + L.acc_w);
  h->acc_ew = reinterpret_cast<double*>(w + L.acc_ew);
  h->eepf = reinterpret_cast<unsigned long long*>(w + L.eepf);
  for (int sp = 0; sp < 2; ++sp) h->fedf[sp] = reinterpret_cast<unsigned long long*>(w + L.fedf[sp]);
  h->fedf_emax[0] = p->eepf_emax_ev;
  h->fedf_emax[1] = fedf_ion_emax(p->rf_voltage_v);
  for (int s = 0; s < 2; ++s) {
    h->sort_cnt[s] = reinterpret_cast<uint32_t*>(w + L.sort_cnt[s]);
    h->sort_tot[s] = reinterpret_cast<uint32_t*>(w + L.sort_tot[s]);
  }
  h->cand = reinterpret_cast<uint32_t*>(w + L.cand);
  h->dq = reinterpret_cast<uint32_t*>(w + L.dq);
  h->sort_blocks = L.sort_blocks;
  h->step = 0;
  h->cur[0] = h->cur[1] = 0;
  h->pcur[0] = h->pcur[1] = 0;
  h->e_decided = 0;
  h->pipeline = 1;
  h->measuring = 0;

  if (hipHostMalloc((void**)&h->report, (report_words(h) + 2) * 8, hipHostMallocDefault) !=
      hipSuccess) {
    delete h;
    return PIC_EHIP;
  }
  h->seen = reinterpret_cast<int64_t*>(h->report + report_words(h));
  h->seen[0] = h->seen[1] = -1;
  h->unseen = 0;
  int st = PIC_OK;
  if (hipMemsetAsync(workspace, 0, L.total, h->stream) != hipSuccess ||
      hipMemcpyAsync(h->cum[0], cum[0].data(), cum[0].size() * 8, hipMemcpyHostToDevice,
                     h->stream) != hipSuccess ||
      hipMemcpyAsync(h->cum[1], cum[1].data(), cum[1].size() * 8, hipMemcpyHostToDevice,
                     h->stream) != hipSuccess ||
      hipMemcpyAsync(h->th_cp, th_cp.data(), th_cp.size() * 8, hipMemcpyHostToDevice,
                     h->stream) != hipSuccess ||
      hipMemcpyAsync(h->th_m, th_m.data(), th_m.size() * 8, hipMemcpyHostToDevice, h->stream) !=
          hipSuccess ||
      hipStreamSynchronize(h->stream) != hipSuccess)
    st = PIC_EHIP;
  if (st) {
    (void)hipHostFree(h->report);
    delete h;
    return st;
  }
  for (int s = 0; s < 2; ++s)
    h->launch[s] = particle_launch_config(s, h->nx, p->eepf_bins, h->num_cu, h->max_tiles[s]);
  h->d.n_x = h->nx;
  h->d.n_tiles_max = (int32_t)(L.max_tiles[0] > L.max_tiles[1] ? L.max_tiles[0] : L.max_tiles[1]);
  h->d.dx = h->dx;
  h->d.dt = h->dt;
  h->d.gas_density = h->ng;
  for (int s = 0; s < 2; ++s) {
    h->d.nu_max[s] = h->numax[s];
    h->d.p_coll[s] = h->pcoll[s];
  }
  *out = h;
  return PIC_OK;
}

int pic_get_derived(const pic_handle* h, pic_derived* d) {
  if (!h || !d) return PIC_EINVAL;
  *d = h->d;
  return PIC_OK;
}

int pic_set_state(pic_handle* h, int species, const double* x, const double* vx, const double* vy,
                  const double* vz, int64_t n, int64_t step) {
  if (!h || species < 0 || species > 1 || n < 0 || step < 0) return PIC_EINVAL;
  if (n > 0 && (!x || !vx || !vy || !vz)) return PIC_EINVAL;
  if (n > h->p.capacity[species]) return PIC_ECAPACITY;
  return replace_state(h, species, n, step, [&](InstallArgs& a) {
    if (on_device(h, x) && on_device(h, vx) && on_device(h, vy) && on_device(h, vz)) {
      a.sx = x;
      a.svx = vx;
      a.svy = vy;
      a.svz = vz;
    } else {
      // x and v_x in place, v_y and v_z through the idle pool buffer
      double* const tmp = reinterpret_cast<double*>(h->pool[species][1 - h->pcur[species]]);
      double* const tmp_z = tmp + h->pcap[species];
      HIP_TRY(hipMemcpyAsync(a.x, x, (size_t)n * 8, hipMemcpyDefault, h->stream));
      HIP_TRY(hipMemcpyAsync(a.vx, vx, (size_t)n * 8, hipMemcpyDefault, h->stream));
      HIP_TRY(hipMemcpyAsync(tmp, vy, (size_t)n * 8, hipMemcpyDefault, h->stream));
      HIP_TRY(hipMemcpyAsync(tmp_z, vz, (size_t)n * 8, hipMemcpyDefault, h->stream));
      a.sx = a.x;
      a.svx = a.vx;
      a.svy = tmp;
      a.svz = tmp_z;
    }
    HIP_TRY(launch_install(a, h->stream));
    return PIC_OK;
  });
}

int pic_load_profile(pic_handle* h, int species, int64_t n, const double* dens, const double* temp_ev,
                     int npts, int64_t step) {
  if (!h || species < 0 || species > 1 || n < 0 || step < 0) return PIC_EINVAL;
  if (npts < 2 || npts > kMaxLoadPoints || (n > 0 && (!dens || !temp_ev))) return PIC_EINVAL;
  if (n > h->p.capacity[species]) return PIC_ECAPACITY;
  return replace_state(h, species, n, step, [&](InstallArgs& p) {
    LoadArgs a{};
    a.dens = dens;
    a.temp = temp_ev;
    a.L = h->L;
    a.h = h->L / (double)(npts - 1);
    a.hh = 0.5 * a.h;
    a.vfac = kQe / h->mass[species];
    a.npts = npts;
    a.species = species;
    a.seed = h->p.seed;
    a.run = h->p.run;
    HIP_TRY(launch_load_profile(a, p, h->stream));
    return PIC_OK;
  });
}

int pic_get_state(pic_handle* h, int species, double* x, double* vx, double* vy, double* vz,
                  int64_t cap, int64_t* n, int64_t* step) {
  if (!h || species < 0 || species > 1 || !n) return PIC_EINVAL;
  const bool arrays = x && vx && vy && vz;
  ReportArgs a = report_args(h);
  double* const* part = h->part[species][h->cur[species]];
  const uint32_t* id = h->pid[species][h->cur[species]];
  const double2* pool = h->pool[species][h->pcur[species]];
  const bool direct = arrays && cap > 0 && on_device(h, x) && on_device(h, vx) &&
                      on_device(h, vy) && on_device(h, vz);
  if (direct) {
    // device arrays are written by the kernel that reports the count
    const ExportArgs e{part[0], part[1], id, pool, {x, vx, vy, vz}, cap, species};
    HIP_TRY(launch_export(e, a, h->stream));
  } else {
    HIP_TRY(launch_report(a, h->stream));
  }
  HIP_TRY(hipStreamSynchronize(h->stream));
  const int64_t cnt = (int64_t)h->report[species == 0 ? R_NE : R_NI];
  *n = cnt;
  saw_count(h, species, cnt);
  if (step) *step = h->step;
  const int st = report_status(h);
  if (st) return st;
  if (cnt > cap) return PIC_ECAPACITY;
  if (cnt > 0 && !arrays) return PIC_EINVAL;
  if (cnt == 0 || direct) return PIC_OK;
  // v_y, v_z in slot order, gathered through the pool indices into the idle
  // pool buffer
  double* const tmp = reinterpret_cast<double*>(h->pool[species][1 - h->pcur[species]]);
  double* const tmp_z = tmp + h->pcap[species];
  HIP_TRY(launch_gather(id, pool, tmp, tmp_z, cnt, h->stream));
  HIP_TRY(hipMemcpyAsync(x, part[0], (size_t)cnt * 8, hipMemcpyDefault, h->stream));
  HIP_TRY(hipMemcpyAsync(vx, part[1], (size_t)cnt * 8, hipMemcpyDefault, h->stream));
  HIP_TRY(hipMemcpyAsync(vy, tmp, (size_t)cnt * 8, hipMemcpyDefault, h->stream));
  HIP_TRY(hipMemcpyAsync(vz, tmp_z, (size_t)cnt * 8, hipMemcpyDefault, h->stream));
  HIP_TRY(hipStreamSynchronize(h->stream));
  return PIC_OK;
}

int pic_step(pic_handle* h, int64_t n_steps) {
  if (!h || n_steps < 0) return PIC_EINVAL;
  if ((h->p.flags & PIC_FLAG_FIXED_E) && !h->field_fixed_set) return PIC_ESTATE;
  while (n_steps > 0) {
    take_counts(h);
    StepShape c;
    bool one_kernel;
    int st = step_route(h, n_steps, &c, &one_kernel);
    if (st) return st;
    int64_t done = n_steps;
    if (one_kernel) {
      st = run_step_kernels(h, n_steps, c, &done);
    } else {
      st = run_passes(h, n_steps);
      h->unseen += n_steps;
    }
    if (!st) st = ask_counts(h);
    if (st) return st;
    n_steps -= done;
  }
  return PIC_OK;
}

int pic_step_many(pic_handle* const* handles, int n, int64_t n_steps, int64_t chunk) {
  if (n < 0 || n_steps < 0 || chunk < 1 || (n > 0 && !handles)) return PIC_EINVAL;
  for (int i = 0; i < n; ++i) {
    if (!handles[i]) return PIC_EINVAL;
    for (int k = 0; k < i; ++k)
      if (handles[k] == handles[i]) return PIC_EINVAL;
  }
  for (int64_t done = 0; done < n_steps; done += chunk) {
    const int64_t m = (n_steps - done < chunk) ? n_steps - done : chunk;
    for (int i = 0; i < n; ++i) {
      const int st = pic_step(handles[i], m);
      if (st) return st;
    }
  }
  return PIC_OK;
}

int pic_batch_workspace_bytes(pic_handle* const* handles, int n, uint64_t* bytes) {
  if (!bytes) return PIC_EINVAL;
  const int v = check_batch_handles(handles, n);
  if (v) return v;
  *bytes = 2 * (uint64_t)batch_half_bytes(n, handles[0]->num_cu);
  return PIC_OK;
}

int pic_batch_create(pic_handle* const* handles, int n, void* workspace, uint64_t workspace_bytes,
                     pic_batch** out) {
  if (!out) return PIC_EINVAL;
  *out = nullptr;
  const int v = check_batch_handles(handles, n);
  if (v) return v;
  const int chunk = batch_chunk_steps(n);
  const size_t half = batch_half_bytes(n, handles[0]->num_cu);
  if (!workspace || workspace_bytes < 2 * half || ((uintptr_t)workspace % kAlign) != 0)
    return PIC_EINVAL;
  pic_batch* b = new (std::nothrow) pic_batch();
  if (!b) return PIC_EINVAL;
  b->hs.assign(handles, handles + n);
  b->stream = handles[0]->stream;
  b->chunk = chunk;
  b->slot = 0;
  b->num_cu = handles[0]->num_cu;
  b->nx_max = b->nbins_max = 0;
  for (pic_handle* h : b->hs) {
    b->nx_max = h->nx > b->nx_max ? h->nx : b->nx_max;
    b->nbins_max = h->p.eepf_bins > b->nbins_max ? h->p.eepf_bins : b->nbins_max;
  }
  b->variants = false;
  for (pic_handle* h : b->hs)
    if (h->p.flags & (PIC_FLAG_ANISO_ELASTIC | PIC_FLAG_OPAL_SHARING)) b->variants = true;
  int64_t tiles[2] = {0, 0};
  for (pic_handle* h : b->hs)
    for (int sp = 0; sp < 2; ++sp) tiles[sp] += h->max_tiles[sp];
  b->passes = batch_launch_config(b->nx_max, b->nbins_max, b->num_cu, tiles);
  for (int k = 0; k < 4; ++k) b->step_fit[k / 2][k % 2] = 0;
  b->counts = nullptr;
  b->unseen = 0;
  for (int k = 0; k < 2; ++k) {
    b->dev[k] = static_cast<unsigned char*>(workspace) + k * half;
    b->host[k] = nullptr;
    b->copied[k] = nullptr;
  }
  bool ok = true;
  for (int k = 0; k < 2 && ok; ++k) {
    ok = hipHostMalloc((void**)&b->host[k], half, hipHostMallocDefault) == hipSuccess &&
         hipEventCreateWithFlags(&b->copied[k], hipEventDisableTiming) == hipSuccess;
  }
  ok = ok && hipHostMalloc((void**)&b->counts, (size_t)n * 2 * sizeof(int64_t),
                           hipHostMallocDefault) == hipSuccess;
  if (!ok) {
    pic_batch_free(b);
    return PIC_EHIP;
  }
  for (int i = 0; i < 2 * n; ++i) b->counts[i] = -1;
  *out = b;
  return PIC_OK;
}

int pic_batch_step(pic_batch* b, int64_t n_steps) {
  if (!b || n_steps < 0) return PIC_EINVAL;
  for (pic_handle* h : b->hs)
    if ((h->p.flags & PIC_FLAG_FIXED_E) && !h->field_fixed_set) return PIC_ESTATE;
  while (n_steps > 0) {
    // the route and the tiles are looked at again every so many steps
    const int64_t m = n_steps < kLookSteps ? n_steps : kLookSteps;
    take_batch_counts(b);
    StepShape c;
    int st = batch_plan_shape(b, &c);
    if (st) return st;
    st = batch_kernel_pays(b, c, m) ? batch_step_kernels(b, m, c) : batch_passes(b, m);
    if (st) return st;
    n_steps -= m;
  }
  return PIC_OK;
}

void pic_batch_free(pic_batch* b) {
  if (!b) return;
  (void)hipStreamSynchronize(b->stream);
  for (int k = 0; k < 2; ++k) {
    if (b->host[k]) (void)hipHostFree(b->host[k]);
    if (b->copied[k]) (void)hipEventDestroy(b->copied[k]);
  }
  if (b->counts) (void)hipHostFree(b->counts);
  delete b;
}

int pic_sync(pic_handle* h) {
  if (!h) return PIC_EINVAL;
  return latched(h);
}

int pic_set_field(pic_handle* h, const double* E) {
  if (!h || !E) return PIC_EINVAL;
  if (!(h->p.flags & PIC_FLAG_FIXED_E)) return PIC_ESTATE;
  for (int b = 0; b < 2; ++b)
    HIP_TRY(hipMemcpyAsync(h->Ebuf[b], E, (size_t)h->nx * 8, hipMemcpyDefault, h->stream));
  HIP_TRY(hipStreamSynchronize(h->stream));
  h->field_fixed_set = 1;
  return PIC_OK;
}

int pic_get_field(pic_handle* h, double* rho, double* phi, double* E, int64_t* deposit_e,
                  int64_t* deposit_i) {
  if (!h) return PIC_EINVAL;
  const size_t b = (size_t)h->nx * 8;
  ReportArgs a = report_args(h);
  const void* src[5] = {h->rho, h->phi, h->Ebuf[h->e_last], dep_buf(h, 0, 0), dep_buf(h, 1, 0)};
  void* const dst[5] = {rho, phi, E, deposit_e, deposit_i};
  for (int k = 0; k < 5; ++k) {
    const bool host = dst[k] && on_host(dst[k]);
    if (dst[k] && !host) HIP_TRY(hipMemcpyAsync(dst[k], src[k], b, hipMemcpyDefault, h->stream));
    a.src[k] = src[k];
    a.n[k] = host ? h->nx : 0;
  }
  const int st = read_report(h, a);
  if (st) return st;
  const uint64_t* r = h->report + R_ARRAYS;
  for (int k = 0; k < 5; ++k)
    if (a.n[k]) {
      std::memcpy(dst[k], r, b);
      r += h->nx;
    }
  return report_status(h);
}

int pic_measure(pic_handle* h, int on) {
  if (!h) return PIC_EINVAL;
  h->measuring = on ? 1 : 0;
  return PIC_OK;
}

int pic_moments(pic_handle* h, pic_moments_out* out, int reset) {
  if (!h || !out) return PIC_EINVAL;
  const int nx = h->nx, nb = h->p.eepf_bins;
  ReportArgs a = report_args(h);
  const void* src[5] = {h->acc_ne, h->acc_ni, h->acc_w, h->acc_ew, h->eepf};
  for (int k = 0; k < 5; ++k) {
    a.src[k] = src[k];
    a.n[k] = k < 4 ? nx : nb;
  }
  const int st = read_report(h, a);
  if (st) return st;
  const int64_t msteps = (int64_t)h->report[R_MSTEPS];
  const double* ne = reinterpret_cast<const double*>(h->report + R_ARRAYS);
  const double *ni = ne + nx, *w = ni + nx, *ew = w + nx;
  const uint64_t* hist = h->report + R_ARRAYS + 4 * (size_t)nx;
  for (int j = 0; j < nx; ++j) {
    if (out->n_e) out->n_e[j] = msteps ? ne[j] / (double)msteps : 0.0;
    if (out->n_i) out->n_i[j] = msteps ? ni[j] / (double)msteps : 0.0;
    if (out->mean_energy_e) out->mean_energy_e[j] = w[j] > 0.0 ? ew[j] / w[j] : 0.0;
  }
  if (out->eepf) {
    unsigned long long tot = 0;
    for (int b = 0; b < nb; ++b) tot += hist[b];
    for (int b = 0; b < nb; ++b) {
      const double eb = ((double)b + 0.5) * h->eepf_de;
      out->eepf[b] = tot ? (double)hist[b] / ((double)tot * std::sqrt(eb) * h->eepf_de) : 0.0;
    }
  }
  out->steps_averaged = msteps;
  if (reset) {
    ClearArgs c{{reinterpret_cast<uint64_t*>(h->acc_ne), reinterpret_cast<uint64_t*>(h->acc_ni),
                 reinterpret_cast<uint64_t*>(h->acc_w), reinterpret_cast<uint64_t*>(h->acc_ew),
                 reinterpret_cast<uint64_t*>(h->eepf), reinterpret_cast<uint64_t*>(h->fedf[0]),
                 reinterpret_cast<uint64_t*>(h->fedf[1]),
                 reinterpret_cast<uint64_t*>(h->ctl->wall_hits),
                 reinterpret_cast<uint64_t*>(&h->ctl->msteps), nullptr},
                {nx, nx, nx, nx, nb, 2 * nb, 2 * nb, 13, 1, 0}};
    static_assert(offsetof(DevCtl, ioniz_meas) - offsetof(DevCtl, wall_hits) == 12 * 8,
                  "the electrode sums lie next to each other");
    HIP_TRY(launch_clear(c, h->stream));
  }
  return report_status(h);
}

int pic_wall_moments(pic_handle* h, pic_wall_out* out) {
  if (!h || !out) return PIC_EINVAL;
  const int nb = h->p.eepf_bins;
  ReportArgs a = report_args(h);
  for (int sp = 0; sp < 2; ++sp) {
    a.src[sp] = h->fedf[sp];
    a.n[sp] = 2 * nb;
  }
  const int st = read_report(h, a);
  if (st) return st;
  const uint64_t* hist[2] = {h->report + R_ARRAYS, h->report + R_ARRAYS + 2 * (size_t)nb};
  uint64_t hits[2][2], absd[2][2];
  double esum[2][2];
  std::memcpy(hits, h->report + R_HITS, sizeof(hits));
  std::memcpy(absd, h->report + R_ABSORBED, sizeof(absd));
  std::memcpy(esum, h->report + R_ESUM, sizeof(esum));
  const uint64_t ioniz = h->report[R_IONIZ];
  const int64_t msteps = (int64_t)h->report[R_MSTEPS];
  // particles per m^2 per s over the measured time msteps * dt
  const double per = msteps ? h->p.weight / (h->p.area_m2 * (double)msteps * h->dt) : 0.0;
  for (int sp = 0; sp < 2; ++sp) {
    const double de = h->fedf_emax[sp] / (double)nb;
    out->fedf_emax_ev[sp] = h->fedf_emax[sp];
    for (int w = 0; w < 2; ++w) {
      out->arrivals[sp][w] = (int64_t)hits[sp][w];
      out->absorbed[sp][w] = (int64_t)absd[sp][w];
      out->flux[sp][w] = per * (double)hits[sp][w];
      out->absorbed_flux[sp][w] = per * (double)absd[sp][w];
      out->mean_energy_ev[sp][w] = hits[sp][w] ? esum[sp][w] / (double)hits[sp][w] : 0.0;
      double* f = out->fedf[sp][w];
      if (!f) continue;
      unsigned long long tot = 0;
      for (int b = 0; b < nb; ++b) tot += hist[sp][(size_t)w * nb + b];
      for (int b = 0; b < nb; ++b)
        f[b] = tot ? (double)hist[sp][(size_t)w * nb + b] / ((double)tot * de) : 0.0;
    }
  }
  out->fedf_bins = nb;
  out->ionizations = (int64_t)ioniz;
  out->ionization_rate = per * (double)ioniz;
  out->steps_averaged = msteps;
  return report_status(h);
}

int pic_get_monitors(pic_handle* h, pic_monitors* out) {
  if (!h || !out) return PIC_EINVAL;
  const int nx = h->nx;
  ReportArgs a = report_args(h);
  const void* src[3] = {h->acc_ne, h->acc_w, h->acc_ew};
  for (int k = 0; k < 3; ++k) {
    a.src[k] = src[k];
    a.n[k] = nx;
  }
  const int st = read_report(h, a);
  if (st) return st;
  const int64_t msteps = (int64_t)h->report[R_MSTEPS];
  double* ne = reinterpret_cast<double*>(h->report + R_ARRAYS);
  const double *w = ne + nx, *ew = w + nx;
  out->steps_averaged = msteps;
  out->p_coll[0] = h->pcoll[0];
  out->p_coll[1] = h->pcoll[1];
  double nmax = 0.0;
  for (int j = 0; j < nx; ++j) {
    ne[j] = msteps ? ne[j] / (double)msteps : 0.0;
    nmax = ne[j] > nmax ? ne[j] : nmax;
  }
  // centre values: the middle node, or the mean of the two middle nodes
  const int j0 = (nx - 1) / 2, j1 = nx / 2;
  const double nc = 0.5 * (ne[j0] + ne[j1]);
  const double e0 = w[j0] > 0.0 ? ew[j0] / w[j0] : 0.0;
  const double e1 = w[j1] > 0.0 ? ew[j1] / w[j1] : 0.0;
  const double ec = 0.5 * (e0 + e1);
  out->n_e_max = nmax;
  out->n_e_center = nc;
  out->mean_energy_center_ev = ec;
  out->omega_pe_dt = std::sqrt(nmax * kQe * kQe / (kEps0 * kMe)) * h->dt;
  const double te = (2.0 / 3.0) * ec;  // eV
  out->lambda_d_m = nc > 0.0 ? std::sqrt(kEps0 * te / (kQe * nc)) : 0.0;
  out->dx_over_lambda_d = out->lambda_d_m > 0.0 ? h->dx / out->lambda_d_m : 0.0;
  out->n_d = nc * h->p.area_m2 * out->lambda_d_m / h->p.weight;
  return report_status(h);
}

int pic_get_counters(pic_handle* h, int64_t* counters) {
  if (!h || !counters) return PIC_EINVAL;
  ReportArgs a = report_args(h);
  a.counters = 1;
  const int st = read_report(h, a);
  if (st) return st;
  std::memcpy(counters, h->report + R_COUNTERS, NCOUNTERS * 8);
  return report_status(h);
}

int pic_get_decisions(pic_handle* h, int species, uint8_t* codes, int64_t cap, int64_t* n) {
  if (!h || species < 0 || species > 1 || !n) return PIC_EINVAL;
  if (!(h->p.flags & PIC_FLAG_RECORD)) return PIC_ESTATE;
  const int st = read_report(h, report_args(h));
  if (st) return st;
  const int64_t cnt = (int64_t)h->report[species == 0 ? R_NCODES_E : R_NCODES_I];
  *n = cnt;
  if (cnt > cap) return PIC_ECAPACITY;
  if (cnt > 0) {
    if (!codes) return PIC_EINVAL;
    HIP_TRY(hipMemcpyAsync(codes, h->codes[species][h->csel[species] ^ 1], (size_t)cnt,
                           hipMemcpyDefault, h->stream));
    HIP_TRY(hipStreamSynchronize(h->stream));
  }
  return report_status(h);
}

int pic_set_launch(pic_handle* h, int decide_wg_per_cu, int emit_wg_per_cu) {
  if (!h || decide_wg_per_cu < 1 || emit_wg_per_cu < 1) return PIC_EINVAL;
  for (int s = 0; s < 2; ++s) particle_launch_set(h->launch[s], h->num_cu, decide_wg_per_cu, emit_wg_per_cu);
  h->step_wg = emit_wg_per_cu;
  return PIC_OK;
}

int pic_set_decide_block(pic_handle* h, int threads) {
  if (!h || (threads != kDecideBlocks[0] && threads != kDecideBlocks[1])) return PIC_EINVAL;
  for (int s = 0; s < 2; ++s)
    if (!particle_launch_block(h->launch[s], h->num_cu, threads)) return PIC_EINVAL;
  return PIC_OK;
}

int pic_set_pipeline(pic_handle* h, int on) {
  if (!h || on < 0 || on > 1) return PIC_EINVAL;
  h->pipeline = on;
  return PIC_OK;
}

int pic_tune(pic_handle* h, int64_t steps_per_trial, int* decide_wg_per_cu, int* emit_wg_per_cu) {
  if (!h || steps_per_trial < 1) return PIC_EINVAL;
  // time one kernel of the electron pass over steps_per_trial steps with
  // events around every particle kernel, without disturbing the caller's
  // accumulated timers
  const int level = h->timing;
  auto trial = [&](int timer, double* us) -> int {
    int st = timer_collect(h);
    if (st) return st;
    const double ms0 = h->t_ms[timer];
    const int64_t n0 = h->t_n[timer];
    h->timing = 2;
    st = pic_step(h, steps_per_trial);
    if (!st) st = timer_collect(h);
    h->timing = level;
    if (st) return st;
    const int64_t n = h->t_n[timer] - n0;
    *us = n ? 1e3 * (h->t_ms[timer] - ms0) / (double)n : 0.0;
    h->t_ms[timer] = ms0;
    h->t_n[timer] = n0;
    return PIC_OK;
  };
  // the shape of the kernels that are timed; one-kernel steps keep theirs
  auto set = [&](int kd, int ke) {
    for (int s = 0; s < 2; ++s) particle_launch_set(h->launch[s], h->num_cu, kd, ke);
  };
  const PartLaunch launch0[2] = {h->launch[0], h->launch[1]};
  const PartLaunch& c = launch0[0];
  int kd = c.bpc_decide[0], ke = c.bpc_emit;
  int st = PIC_OK;
  double best = -1.0;
  for (int k = 1; k <= c.bpc_decide[0] && !st; ++k) {
    set(k, c.bpc_emit);
    double us = 0.0;
    st = trial(PIC_TIMER_E_DECIDE, &us);
    if (!st && (best < 0.0 || us < best)) {
      best = us;
      kd = k;
    }
  }
  best = -1.0;
  for (int k = 1; k <= c.bpc_emit && !st; ++k) {
    set(kd, k);
    double us = 0.0;
    st = trial(PIC_TIMER_E_EMIT, &us);
    if (!st && (best < 0.0 || us < best)) {
      best = us;
      ke = k;
    }
  }
  if (st) {
    for (int s = 0; s < 2; ++s) h->launch[s] = launch0[s];
    return st;
  }
  set(kd, ke);
  if (decide_wg_per_cu) *decide_wg_per_cu = kd;
  if (emit_wg_per_cu) *emit_wg_per_cu = ke;
  return latched(h);
}

int pic_tune_pass(pic_handle* h, int64_t steps_per_trial, pic_pass_trial* trials, int max_trials,
                  int* n_trials, int* best) {
  if (!h || steps_per_trial < 1 || max_trials < 0 || (max_trials > 0 && !trials)) return PIC_EINVAL;
  // what changes along the way, given back on an error
  const int level = h->timing, pipeline0 = h->pipeline, step_wg0 = h->step_wg;
  const PartLaunch launch0[2] = {h->launch[0], h->launch[1]};
  hipEvent_t ev[2] = {nullptr, nullptr};
  // every candidate alike: the whole steps between two events, without the
  // pass timers (which would change the schedule)
  auto trial = [&](double* us) -> int {
    float ms = 0.f;
    if (hipEventRecord(ev[0], h->stream) != hipSuccess) return PIC_EHIP;
    const int st = pic_step(h, steps_per_trial);
    if (st) return st;
    if (hipEventRecord(ev[1], h->stream) != hipSuccess ||
        hipEventSynchronize(ev[1]) != hipSuccess ||
        hipEventElapsedTime(&ms, ev[0], ev[1]) != hipSuccess)
      return PIC_EHIP;
    *us = 1e3 * (double)ms / (double)steps_per_trial;
    return PIC_OK;
  };
  const PartLaunch& c = launch0[0];
  int n = 0, ib = -1;
  pic_pass_trial bestt{};
  auto run = [&](int pipe, int db, int kd, int ke, double* us) -> int {
    h->pipeline = pipe;
    int st = pic_set_decide_block(h, db);
    if (!st) st = pic_set_launch(h, kd, ke);
    if (st) return st;
    pic_pass_trial t{pipe, db, kd, ke, 0.0};
    st = trial(&t.us_per_step);
    if (st) return st;
    if (n < max_trials) trials[n] = t;
    if (ib < 0 || t.us_per_step < bestt.us_per_step) {
      ib = n;
      bestt = t;
    }
    ++n;
    *us = t.us_per_step;
    return PIC_OK;
  };
  int st = timer_collect(h);
  if (!st && (hipEventCreate(&ev[0]) != hipSuccess || hipEventCreate(&ev[1]) != hipSuccess))
    st = PIC_EHIP;
  h->timing = 0;
  double us = 0.0;
  // pipelined: the workgroups per CU of the one-kernel step, or where the
  // passes are taken of the fused emit (whose decide pass runs only on the
  // steps that cannot be pipelined, at the default size and the most workgroups
  // that fit)
  const int kd_max = c.bpc_decide_by[0][0];
  h->pipeline = 1;
  StepShape shape;
  bool one_kernel = false;
  if (!st) st = step_route(h, steps_per_trial, &shape, &one_kernel);
  const int k_max = one_kernel ? shape.fit : c.bpc_emit_decide;
  for (int k = 1; k <= k_max && !st; ++k) st = run(1, kDecideBlocks[0], kd_max, k, &us);
  // unpipelined: each compiled decide size at each of its shapes, then each
  // emit shape at the best decide
  int db_best = kDecideBlocks[0], kd_best = kd_max;
  double kd_us = -1.0;
  for (int b = 0; b < 2 && !st; ++b) {
    for (int k = 1; k <= c.bpc_decide_by[b][0] && !st; ++k) {
      st = run(0, kDecideBlocks[b], k, c.bpc_emit, &us);
      if (!st && (kd_us < 0.0 || us < kd_us)) {
        kd_us = us;
        db_best = kDecideBlocks[b];
        kd_best = k;
      }
    }
  }
  for (int k = 1; k < c.bpc_emit && !st; ++k) st = run(0, db_best, kd_best, k, &us);
  for (hipEvent_t v : ev)
    if (v) (void)hipEventDestroy(v);
  h->timing = level;
  if (st) {
    h->pipeline = pipeline0;
    h->step_wg = step_wg0;
    for (int s = 0; s < 2; ++s) h->launch[s] = launch0[s];
    return st;
  }
  h->pipeline = bestt.pipeline;
  pic_set_decide_block(h, bestt.decide_block);
  pic_set_launch(h, bestt.decide_wg_per_cu, bestt.emit_wg_per_cu);
  if (n_trials) *n_trials = n;
  if (best) *best = ib;
  return latched(h);
}

int pic_timing(pic_handle* h, int level) {
  if (!h || level < 0 || level > 2) return PIC_EINVAL;
  h->timing = level;
  return PIC_OK;
}

int pic_get_timing(pic_handle* h, double* ms, int64_t* launches, int reset) {
  if (!h) return PIC_EINVAL;
  const int st = timer_collect(h);
  if (st) return st;
  for (int i = 0; i < PIC_NTIMERS; ++i) {
    if (ms) ms[i] = h->t_ms[i];
    if (launches) launches[i] = h->t_n[i];
    if (reset) {
      h->t_ms[i] = 0.0;
      h->t_n[i] = 0;
    }
  }
  return PIC_OK;
}

void pic_free(pic_handle* h) {
  if (!h) return;
  (void)hipStreamSynchronize(h->stream);
  for (hipEvent_t e : h->ev_pool) (void)hipEventDestroy(e);
  (void)hipHostFree(h->report);
  delete h;
}

int pic_selftest_philox(const uint32_t* ctr, const uint32_t* key, uint32_t* out, int64_t n,
                        void* stream) {
  if (n < 0 || !key || (n > 0 && (!ctr || !out))) return PIC_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  HIP_TRY(launch_selftest_philox(ctr, key[0], key[1], out, n, s));
  HIP_TRY(hipStreamSynchronize(s));
  return PIC_OK;
}

int pic_selftest_sqrt(const double* in, double* out, int64_t n, void* stream) {
  if (n < 0 || (n > 0 && (!in || !out))) return PIC_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  HIP_TRY(launch_selftest_sqrt(in, out, n, s));
  HIP_TRY(hipStreamSynchronize(s));
  return PIC_OK;
}

int pic_selftest_copy(const double* in, double* out, int64_t n, void* stream) {
  if (n < 0 || (n & 1) || (n > 0 && (!in || !out))) return PIC_EINVAL;
  if (((uintptr_t)in | (uintptr_t)out) & 15) return PIC_EINVAL;
  HIP_TRY(launch_selftest_copy(in, out, n, (hipStream_t)stream));
  return PIC_OK;
}

}  // extern "C"
