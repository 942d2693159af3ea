// qed_step.hip -- the per-step kernels of the QED step (Sec. IV.H adaptive event generator
// of Gonoskov et al., arXiv:1412.6426, with the Sec. V.A pair generator).
//
// One step is five launches on the caller's stream, up to eight in its other forms (plus three
// per same-step generation):
//   prep     (1 + k wgs)    snapshot live counts, particle prefix sums over the
//                           (instance, species) segments, space-independent fields at t_n,
//                           zero the stats record and the arenas' count matrices;
//   leptons  (persistent)   electrons and positrons: push, chi, emission; emitted photons
//                           go to the wavefront's share of the photon arena;
//   photons  (persistent)   photons: push, chi_gamma, pair-rate bound; draws below the
//                           bound go to the wavefront's candidate list (leptons and photons
//                           are workgroups of one launch, except with same-step children, a
//                           generator factor, its reverse mode, events around them, or
//                           workgroups of other sizes than 256) for
//   exact    (persistent)   the exact pair decision; pair records go to the pair arena;
//   scan     (2 wgs/instance) arena counts -> store offsets, instance counts raised and
//                           clamped to the capacities;
//   copy     (1 wave/source wave) arena records -> photon, electron, positron stores;
//   reduce   (1 wave per eight fields of 128 workgroups) per-workgroup partial stats -> the
//                           stats record (status bits set with the counters they report);
//   finalize (1 workgroup)  clamp counts, step index + 1.
// Where the copy is the step's last producer (arenas on, no same-step children), its launch
// also takes the reduce jobs and the step index.
// Children land after the step-start counts, so they are first processed at step n+1.
//
// Work distribution: the particles alive at the step start form one index space per kernel
// (segments of all instances laid end to end).  Each wavefront owns fixed chunks of it --
// no queue, no atomics -- and keeps its 64 lanes busy by refilling any lane whose particle
// has finished all of its sub-steps from the next particles of its chunk ("per-wavefront
// work queue"): one wavefront iteration advances every active lane by one sub-step, so
// lanes with n_sub = 1 and n_sub = 20 share a wavefront without idling.
//
// Appends: a wavefront writes the children it creates into its own share of an arena in
// the workspace (ballot + prefix popcount for the positions, no shared counter) and tallies
// them per instance; a scan per instance turns the tallies into store offsets and a copy
// kernel writes the children to the stores in (instance, wavefront, creation) order.  A
// device-wide counter takes one atomic per reservation and serialises every wavefront of
// the GPU on one address; the arenas avoid that.  Without arena space (or with more than
// kArenaMaxInstances instances) children are staged per wavefront in LDS and reserved in
// batches of up to 32 with one atomic per (batch, instance, species).  Statistics are
// reduced per workgroup in LDS and written as partials, which the reduce jobs sum.
#include "qed_internal.h"

namespace qedk {

constexpr int kWavesPerBlock = 4;  // launch bound 256 threads
constexpr int kStageCap = 32;      // staged photon children per wavefront
// Particles per chunk for N particles on W wavefronts.  Asked for (d.tile): that.  Else the
// largest of 128, 256 and 512 up to d.most that gives every wavefront a chunk; below that 64,
// one batch of lanes each, so that no wavefront takes two batches in turn beside idle ones; and
// where there are fewer than 64 leptons for each of d.spread wavefronts (one a SIMD; 0 for the
// photons, whose loads want full batches), as few as spread them over all of those.
//
// Chunks are dealt round-robin, so the wavefronts of the GPU read neighbouring pieces of every
// column at any moment (measured faster than one contiguous range per wavefront, which scatters
// the reads over the whole store).  d.most: 128 leptons, whose sub-steps differ (512: 75 against
// 63 ms of lepton kernel on the rotating cascade); 512 photons, in whose chunks several
// batches follow each other in memory (128 / 256 / 512 / 1024: the same job 239 / 225 / 224 / 226
// ms, its photon kernel alone 263 / 256 / 251 / 258 us a launch); 128 photons on a Yee grid,
// where neighbouring wavefronts share the grid's lines (8 times the photons of 10^6 leptons: 1214 /
// 1221 / 1247 / 1256 us a step).
//
// A lepton's sub-steps are a serial chain, and one of a wavefront with few lanes takes 1.3 us
// where a full one, with emissions in nearly every sub-step, takes 3.7.  Against 128 throughout:
// 10^4 electrons in a uniform B 78 to 55 us a step, the lepton kernel of 400 electrons with
// thousands of sub-steps each 5.7 to 3.5 ms.
__device__ __forceinline__ long long chunk_size(long long N, long long W, const Deal& d) {
  if (d.tile > 0) return d.tile;
  if (N >= 128 * W) return d.most == 128 || N < 256 * W ? 128 : N < 512 * W ? 256 : 512;
  if (d.spread <= 0 || N >= 64 * d.spread) return 64;
  const unsigned spread = (unsigned)d.spread;
  const unsigned t = ((unsigned)N + spread - 1u) / spread;
  return t < 1u ? 1 : (long long)t;
}

// ------------------------------------------------------------------------------------
// prep / finalize
// ------------------------------------------------------------------------------------
constexpr int kPrepWaves = 4;  // workgroups of 256
__global__ void __launch_bounds__(256) prep_kernel(StepArgs a, int run_photons) {
  if (blockIdx.x > 0) {
    // workgroups 1.. clear the per-(instance, wavefront) child counts of the arenas and
    // their pool counters
    const long long n1 = a.pa.waves > 0 ? (long long)a.n_inst * a.pa.waves : 0;
    const long long n2 = a.qa.waves > 0 ? (long long)a.n_inst * a.qa.waves : 0;
    const long long stride = (long long)(gridDim.x - 1) * blockDim.x;
    for (long long i = (long long)(blockIdx.x - 1) * blockDim.x + threadIdx.x; i < n1 + n2;
         i += stride) {
      if (i < n1) a.pa.cnt[i] = 0u;
      else a.qa.cnt[i - n1] = 0u;
    }
    if (blockIdx.x == 1 && threadIdx.x == 0) {
      if (a.pa.waves > 0) *a.pa.used = 0u;
      if (a.qa.waves > 0) *a.qa.used = 0u;
    }
    return;
  }
  // Instance by instance per thread: the counts, the fields, and a workgroup scan of the
  // counts into the prefixes (64 instances: 10.4 us a launch, 28.4 with one thread walking them).
  __shared__ long long wl[kPrepWaves], wp[kPrepWaves];
  __shared__ long long s_ns[3];
  WorkHdr* hdr = a.hdr;
  const long long n = *a.d_step;
  const double tn = a.t0 + (double)n * a.dt;
  const bool ok = a.tables->magic == kTableMagic;
  const int lane = (int)(threadIdx.x & 63u), wv = (int)(threadIdx.x >> 6);
  unsigned long long* sw = reinterpret_cast<unsigned long long*>(a.stats);
  for (int w = threadIdx.x; w < (int)(sizeof(qed_stats) / 8); w += blockDim.x) sw[w] = 0ull;
  if (threadIdx.x < 3) s_ns[threadIdx.x] = 0;
  __syncthreads();
  long long carry_l = 0, carry_p = 0, ns[3] = {0, 0, 0};
  for (int i0 = 0; i0 < a.n_inst; i0 += (int)blockDim.x) {
    const int i = i0 + (int)threadIdx.x;
    long long live[3] = {0, 0, 0};
    if (i < a.n_inst) {
      qed_instance& I = a.inst[i];
      if (a.freeze_on_drop && I.dropped > 0) I.frozen = 1;
      const bool off = I.frozen || !ok;
      for (int s = 0; s < 3; ++s) {
        long long c = I.count[s];
        if (c > I.capacity[s]) c = I.capacity[s];
        if (c < 0) c = 0;
        I.count[s] = c;
        live[s] = off ? 0 : c;
        a.n0[i * 3 + s] = live[s];
        ns[s] += live[s];
      }
      double* eb = a.eb + 6 * i;
      const double amp = I.amp;
      if (a.field.kind == QED_FIELD_UNIFORM) {
        for (int d = 0; d < 3; ++d) {
          eb[d] = a.e0[d] * amp;
          eb[3 + d] = a.b0[d] * amp;
        }
      } else if (a.field.kind == QED_FIELD_ROTATING_E) {
        double sph, cph;
        sincos(a.field.omega * tn + a.field.phase, &sph, &cph);
        const double e = a.field.amp * amp;
        eb[0] = e * cph;
        eb[1] = e * sph;
        eb[2] = eb[3] = eb[4] = eb[5] = 0.0;
      }
    }
    // inclusive scans over the workgroup's threads of the lepton and photon counts
    long long xl = live[0] + live[1], xp = run_photons ? live[2] : 0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const long long yl = __shfl_up(xl, o, 64), yp = __shfl_up(xp, o, 64);
      if (lane >= o) {
        xl += yl;
        xp += yp;
      }
    }
    if (lane == 63) {
      wl[wv] = xl;
      wp[wv] = xp;
    }
    __syncthreads();
    long long bl = carry_l, bp = carry_p;
    for (int q = 0; q < kPrepWaves; ++q) {
      if (q < wv) {
        bl += wl[q];
        bp += wp[q];
      }
      carry_l += wl[q];
      carry_p += wp[q];
    }
    __syncthreads();
    if (i < a.n_inst) {
      a.lep_pref[2 * i + 2] = bl + xl;
      a.lep_pref[2 * i + 1] = bl + xl - live[1];
      a.pho_pref[i + 1] = bp + xp;
    }
  }
  for (int s = 0; s < 3; ++s)
    if (ns[s]) atomicAdd(reinterpret_cast<unsigned long long*>(&s_ns[s]), (unsigned long long)ns[s]);
  __syncthreads();
  if (threadIdx.x == 0) {
    a.lep_pref[0] = 0;
    a.pho_pref[0] = 0;
    hdr->lep_total = carry_l;
    hdr->pho_total = carry_p;
    hdr->n_cand = 0ull;
    hdr->step = n;
    hdr->tn = tn;
    hdr->tables_ok = ok ? 1u : 0u;
    a.stats->step = n;
    for (int s = 0; s < 3; ++s) a.stats->n_start[s] = s_ns[s];
    if (!ok) a.stats->status = QED_STATUS_NO_TABLES;
  }
}

__device__ __forceinline__ void stats_add(int64_t* p, unsigned long long v) {
  if (v) atomicAdd(reinterpret_cast<unsigned long long*>(p), v);
}

// Where field f of workgroup b's partial record sits: in groups of kPfGroup fields, the group's
// fields of one workgroup side by side (64 bytes) and the workgroups in turn, so that a
// workgroup stores whole lines and the reduction reads them (a row per field left every
// workgroup 182 stores to as many lines).  The last group is as wide as what is left.
constexpr int kPfGroup = 8;
__device__ __forceinline__ size_t part_index(int f, int b) {
  const int g = f / kPfGroup, w = kPfCount - g * kPfGroup < kPfGroup ? kPfCount - g * kPfGroup : kPfGroup;
  return (size_t)g * kPfGroup * kMaxGridBlocks + (size_t)b * w + (size_t)(f - g * kPfGroup);
}

// Partial-stats reduction: one wavefront per (partial set, group of fields, slice of
// kPfSlice workgroups).  The lepton and generation sets have all kPfCount fields; the photon
// and exact-pair sets only the counters below kPfNsub.  Lane l takes field l % 8 of every
// eighth workgroup of the slice, kPfSlice / 8 independent loads (a wavefront per group over all
// workgroups waited for 256 loads in turn: 36 us a launch against 9.5).  Sums go into the zeroed
// stats record with atomics.
constexpr int kPfSlice = 128;
constexpr int kGroupsAll = (kPfCount + kPfGroup - 1) / kPfGroup;
constexpr int kGroupsCount = (kPfNsub + kPfGroup - 1) / kPfGroup;
__host__ __device__ inline int pf_slices(int grid) { return (grid + kPfSlice - 1) / kPfSlice; }
// Jobs of set `kind` (0 leptons, 1 photons, 2 exact pairs, 3 generations), and of all four.
__host__ __device__ inline int reduce_jobs_of(const StepArgs& a, int kind) {
  return kind == 0   ? kGroupsAll * pf_slices(a.lep_grid)
         : kind == 1 ? kGroupsCount * pf_slices(a.pho_grid)
         : kind == 2 ? kGroupsCount * pf_slices(a.ex_grid)
                     : kGroupsAll * pf_slices(a.gen_grid);
}
inline int reduce_blocks(const StepArgs& a) {  // workgroups of 4 wavefronts
  int n = 0;
  for (int kind = 0; kind < 4; ++kind) n += reduce_jobs_of(a, kind);
  return (n + 3) / 4;
}

// Lepton workgroups that share the leptons, where one launch takes photons too: a.lep_beside of
// them, two per CU, where there are kBeside times as many photons, which then fill the rest of
// each CU, else all that the device holds (the ones past the count are idle).  Only forms that
// hold three per CU have the choice (FP64 in a rotating field, mixed in any uniform one).  us a
// step of 10^6 leptons with two / three per CU, FP64 rotating, mixed rotating, mixed uniform:
//   10^3 photons    114 / 99    106 / 93    131 / 114
//   10^6            131 / 126   121 / 120   150 / 139
//   4 10^6          172 / 169   162 / 169   191 / 189
//   8 10^6          229 / 246   223 / 248   258 / 274
constexpr long long kBeside = 2;
__device__ __forceinline__ int lepton_blocks(const StepArgs& a) {
  return a.lep_beside > 0 && a.hdr->pho_total >= kBeside * a.hdr->lep_total ? a.lep_beside
                                                                            : a.lep_grid;
}

__device__ __forceinline__ int working_blocks_of(long long N, int grid, int wpb, const Deal& d);

__device__ __forceinline__ void reduce_job(const StepArgs& a, int job, int lane) {
  int kind = 0;
  while (kind < 4 && job >= reduce_jobs_of(a, kind)) job -= reduce_jobs_of(a, kind++);
  if (kind == 4) return;
  const int groups = kind == 0 || kind == 3 ? kGroupsAll : kGroupsCount;
  const int g = job % groups, b0 = (job / groups) * kPfSlice;
  const bool pho = kind == 1 || kind == 2;
  // the workgroups that have stored a record: idle ones of the lepton and photon kernels do not
  const int G = kind == 0   ? working_blocks_of(a.hdr->lep_total, lepton_blocks(a), a.wpb, a.lep_deal)
                : kind == 1 ? working_blocks_of(a.hdr->pho_total, a.pho_grid, a.wpb, a.pho_deal)
                : kind == 2 ? a.ex_grid
                            : a.gen_grid;
  if (b0 >= G) return;
  const unsigned long long* part =
      kind == 0 ? a.lep_part : (kind == 1 ? a.pho_part : (kind == 2 ? a.ex_part : a.gen_part));
  const int f = g * kPfGroup + (lane & (kPfGroup - 1));
  const bool mine = f < (pho ? kPfNsub : kPfCount);
  const bool sumd = f == kPfEnergy, maxd = f == kPfMaxP || f == kPfMaxQ;
  qed_stats* st = a.stats;
  unsigned long long v = 0ull;
  double d = 0.0;
  if (mine) {
    constexpr int kLoads = kPfSlice * kPfGroup / 64;
    unsigned long long xs[kLoads];
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int b = b0 + lane / kPfGroup + q * (64 / kPfGroup);
      xs[q] = b < G ? part[part_index(f, b)] : 0ull;
    }
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const unsigned long long x = xs[q];
      if (sumd) d += __longlong_as_double((long long)x);
      else if (maxd) d = fmax(d, __longlong_as_double((long long)x));
      else v += x;
    }
  }
#pragma unroll
  for (int o = 32; o >= kPfGroup; o >>= 1) {
    v += __shfl_xor(v, o, 64);
    const double y = __shfl_xor(d, o, 64);
    d = sumd ? d + y : fmax(d, y);
  }
  if (lane >= kPfGroup || !mine) return;
  if (sumd || maxd) {
    if (d != 0.0) {
      if (sumd) {
        if (!pho) atomicAdd(&st->photon_energy, d);
      } else {
        atomic_max_nonneg((pho || f == kPfMaxQ) ? &st->max_p_pair : &st->max_p_emit, d);
      }
    }
    return;
  }
  if (v == 0ull) return;
  switch (f) {
    case kPfSubsteps: stats_add(&st->substeps, v); break;
    case kPfEvents: stats_add(pho ? &st->pairs : &st->emitted, v); break;
    case kPfSaturated:
      stats_add(&st->saturated, v);
      atomicOr(&st->status, QED_STATUS_SATURATED);
      break;
    case kPfNear: stats_add(&st->near_threshold, v); break;
    case kPfNonfinite:
      stats_add(&st->nonfinite, v);
      atomicOr(&st->status, QED_STATUS_NONFINITE);
      break;
    case kPfNearInt: stats_add(&st->nsub_near_int, v); break;
    case kPfClamped:
      stats_add(&st->nsub_clamped, v);
      atomicOr(&st->status, QED_STATUS_NSUB_CLAMPED);
      break;
    case kPfDropped:
      stats_add(&st->dropped, v);
      atomicOr(&st->status, QED_STATUS_DROPPED);
      break;
    case kPfEarly: stats_add(&st->early_out, v); break;
    case kPfAdv0: stats_add(&st->advanced[pho ? QED_PHOTON : QED_ELECTRON], v); break;
    case kPfAdv1: stats_add(&st->advanced[QED_POSITRON], v); break;
    case kPfWaveIters: stats_add(&st->wave_iters, v); break;
    case kPfLowOcc: stats_add(&st->low_occupancy_iters, v); break;
    case kPfPairs: stats_add(&st->pairs, v); break;
    case kPfChildren: stats_add(&st->children_advanced, v); break;
    case kPfDeferred: stats_add(&st->deferred, v); break;
    case kPfRefined: stats_add(&st->nsub_refined, v); break;
    default:
      if (f >= kPfNsub && f < kPfNsub + QED_NSUB_HIST)
        stats_add(&st->nsub_hist[f - kPfNsub], v);
      else if (f >= kPfHist)
        stats_add(&st->photon_hist[f - kPfHist], v);
  }
}

__global__ void __launch_bounds__(256) reduce_kernel(StepArgs a) {
  const int job = (int)blockIdx.x * (int)(blockDim.x >> 6) + (int)(threadIdx.x >> 6);
  reduce_job(a, job, (int)(threadIdx.x & 63u));
}

// The end of a step whose last launch is not the arena copy: counts clamped to the
// capacities, step + 1.  (The status bits are set where their counters are raised.)
__global__ void __launch_bounds__(256) finalize_kernel(StepArgs a) {
  for (int i = threadIdx.x; i < a.n_inst; i += blockDim.x) {
    qed_instance& I = a.inst[i];
    for (int s = 0; s < 3; ++s)
      if (I.count[s] > I.capacity[s]) I.count[s] = I.capacity[s];
  }
  if (threadIdx.x == 0) *a.d_step = a.hdr->step + 1;
}

// ------------------------------------------------------------------------------------
// shared pieces of the persistent kernels
// ------------------------------------------------------------------------------------
// Field modes the persistent kernels are specialised for.
enum FieldMode : int {
  kFieldEB = 0,     // space-independent E and B, evaluated once per instance (uniform field)
  kFieldE = 1,      // space-independent E, B = 0 (rotating electric field)
  kFieldLocal = 2   // evaluated at each particle (CP standing wave, Yee-grid CIC)
};

// Per-lane accumulators (few, to keep registers for the hot path); wavefront-uniform
// counts (sub-steps, events, particles advanced) are kept in scalar registers, and rare
// events (saturation, non-finite values, near-threshold decisions, clamps, drops) go
// straight into the workgroup's LDS record.
struct BlockStats;
__device__ __forceinline__ void block_count(BlockStats& bs, int field);

struct LaneCounters {
  BlockStats* bs = nullptr;
  int early = 0, subs = 0;
  double energy = 0.0, maxp = 0.0;

  // One decision r2 < P.  `fold`: P counts for the largest probability of the step (every
  // emission decision; only the pair decisions that make a pair, which include every P >= 1).
  // One test covers what is rare: P >= 1, a P that is no number, and a near tie.
  __device__ __forceinline__ void note(double P, double r2, bool fold = true) {
    const bool plain = P < 1.0;
    if (fold) maxp = plain ? fmax(maxp, P) : maxp;
    if (!plain || fabs(r2 - P) < kNearThreshold) {
      if (!isfinite(P)) {
        block_count(*bs, kPfNonfinite);
        return;
      }
      if (!plain) {
        if (fold) maxp = fmax(maxp, P);
        block_count(*bs, kPfSaturated);
      }
      if (fabs(r2 - P) < kNearThreshold) block_count(*bs, kPfNear);
    }
  }
};

// Wavefront-uniform counts.
struct WaveCounters {
  long long substeps = 0, events = 0, adv0 = 0, adv1 = 0, wave_iters = 0, low_occ = 0;
  long long pairs = 0, children = 0, deferred = 0;  // same-step processing
};

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Workgroup-level partial stats in LDS.
struct BlockStats {
  unsigned long long w[kPfCount];
  double energy, maxp, maxq;  // maxq: pair decisions of a kernel that also has emissions
};

__device__ __forceinline__ void block_count(BlockStats& bs, int field) {
  atomicAdd(&bs.w[field], 1ull);
}

// Sub-step refinement (Sec. IV.H asks every sub-interval to satisfy Eq. (29)): a sub-step of
// length h that ends in the state (chi, gamma^2 = 1 + p2) is taken again at half the length
// if h > dt_q there, i.e. if hs3 (chi / eps_r)^2 > gamma^2 with
// hs3 = eps_r^2 (h / (kappa 28 pi eps_r))^3 -- unless that would make more than QED_NSUB_MAX
// sub-steps (then it is kept and counted as clamped).  h / dt_q within 1e-12 of 1 is counted
// with the near-integer sub-step ratios.
__device__ __forceinline__ bool refine_substep(const MathTab& mt, double hs3, const Kin& kn,
                                               double h, double eps_r, double inv_lep_scale,
                                               int k, int left, BlockStats& bs) {
  const double lhs = hs3 * kn.c2, rhs = 1.0 + kn.p2;
  if (fabs(lhs - rhs) <= 4e-12 * rhs &&
      fabs(substep_ratio_lepton(mt, h, kn, eps_r, inv_lep_scale) - 1.0) <= 1e-12)
    block_count(bs, kPfNearInt);
  if (!(lhs > rhs)) return false;
  if (k + 2 * left > QED_NSUB_MAX) {
    block_count(bs, kPfClamped);
    return false;
  }
  block_count(bs, kPfRefined);
  return true;
}

__device__ __forceinline__ void block_stats_init(BlockStats& bs) {
  for (int i = threadIdx.x; i < kPfCount; i += blockDim.x) bs.w[i] = 0ull;
  if (threadIdx.x == 0) {
    bs.energy = 0.0;
    bs.maxp = 0.0;
    bs.maxq = 0.0;
  }
}

// Wave totals of the counters into the workgroup's LDS record; `pc` holds the pair decisions
// of a kernel that also makes emission decisions (their largest probability is kept apart).
__device__ void wave_to_block(BlockStats& bs, const LaneCounters& c, const WaveCounters& wc,
                              const LaneCounters* pc = nullptr) {
  const long long early = wave_sum((long long)c.early);
  const long long subs = wave_sum((long long)c.subs);
  const double en = wave_sum(c.energy);
  const double mp = wave_max(c.maxp);
  const double mq = pc ? wave_max(pc->maxp) : 0.0;
  if (lane_id() == 0) {
    const long long vals[10] = {wc.substeps + subs, wc.events, wc.adv0, wc.adv1,
                                wc.wave_iters, wc.low_occ, early, wc.pairs, wc.children,
                                wc.deferred};
    const int fields[10] = {kPfSubsteps, kPfEvents, kPfAdv0, kPfAdv1, kPfWaveIters, kPfLowOcc,
                            kPfEarly, kPfPairs, kPfChildren, kPfDeferred};
    for (int i = 0; i < 10; ++i)
      if (vals[i]) atomicAdd(&bs.w[fields[i]], (unsigned long long)vals[i]);
    if (en != 0.0) atomicAdd(&bs.energy, en);
    if (mp > 0.0)
      atomicMax(reinterpret_cast<unsigned long long*>(&bs.maxp),
                (unsigned long long)__double_as_longlong(mp));
    if (mq > 0.0)
      atomicMax(reinterpret_cast<unsigned long long*>(&bs.maxq),
                (unsigned long long)__double_as_longlong(mq));
  }
}

// After a __syncthreads: store the first `fields` fields of the workgroup's record.
__device__ __forceinline__ void block_stats_store(const BlockStats& bs, unsigned long long* part,
                                                  int fields, int block) {
  for (int i = threadIdx.x; i < fields; i += blockDim.x) {
    unsigned long long v = bs.w[i];
    if (i == kPfEnergy) v = (unsigned long long)__double_as_longlong(bs.energy);
    if (i == kPfMaxP) v = (unsigned long long)__double_as_longlong(bs.maxp);
    if (i == kPfMaxQ) v = (unsigned long long)__double_as_longlong(bs.maxq);
    part[part_index(i, block)] = v;
  }
}

// The same, added to what earlier launches of the kernel stored (first: store).
__device__ __forceinline__ void block_stats_accumulate(const BlockStats& bs,
                                                       unsigned long long* part, bool first) {
  for (int i = threadIdx.x; i < kPfCount; i += blockDim.x) {
    const size_t at = part_index(i, (int)blockIdx.x);
    const unsigned long long old = first ? 0ull : part[at];
    unsigned long long v;
    if (i == kPfEnergy) {
      v = (unsigned long long)__double_as_longlong(
          bs.energy + (first ? 0.0 : __longlong_as_double((long long)old)));
    } else if (i == kPfMaxP || i == kPfMaxQ) {
      const double m = i == kPfMaxP ? bs.maxp : bs.maxq;
      v = (unsigned long long)__double_as_longlong(
          first ? m : fmax(m, __longlong_as_double((long long)old)));
    } else {
      v = bs.w[i] + old;
    }
    part[at] = v;
  }
}

// Append one child per flagged lane to species SP of the lane's instance: one ballot, a
// prefix popcount and one atomic reservation per instance present among the flagged lanes.
// write(store, slot) fills the child's columns.  Must be called by all 64 lanes.
template <int SP, class Writer>
__device__ __forceinline__ void wave_append(const StepArgs& a, bool flag, int inst,
                                            LaneCounters& cnt, Writer&& write) {
  uint64_t m = wave_ballot(flag);
  const uint64_t below = lanes_below();
  while (m) {
    const int leader = __ffsll((unsigned long long)m) - 1;
    const int li = wave_bcast(inst, leader);
    const bool mine = flag && inst == li;
    const uint64_t same = wave_ballot(mine);
    long long base = 0;
    if (lane_id() == leader)
      base = (long long)atomicAdd(reinterpret_cast<unsigned long long*>(&a.inst[li].count[SP]),
                                  (unsigned long long)__popcll(same));
    base = wave_bcast(base, leader);
    const long long cap = a.inst[li].capacity[SP];
    const long long pos = base + __popcll(same & below);
    const bool fits = pos < cap;
    if (mine && fits) write(a.sp[SP], a.inst[li].base[SP] + pos);
    // children beyond the capacity are dropped and counted, once per wavefront
    const uint64_t lost = wave_ballot(mine && !fits);
    if (lost != 0 && lane_id() == leader) {
      atomicAdd(reinterpret_cast<unsigned long long*>(&a.inst[li].dropped),
                (unsigned long long)__popcll(lost));
      atomicAdd(&cnt.bs->w[kPfDropped], (unsigned long long)__popcll(lost));
    }
    m &= ~same;
  }
}

// A wavefront-uniform 64-bit value moved to scalar registers (lane 0's copy).
__device__ __forceinline__ long long wave_uniform(long long v) {
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)v);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((unsigned long long)v >> 32));
  return (long long)(((unsigned long long)hi << 32) | lo);
}

__device__ __forceinline__ double wave_uniform(double v) {
  return __longlong_as_double(wave_uniform((long long)__double_as_longlong(v)));
}
__device__ __forceinline__ V3 wave_uniform(const V3& v) {
  return {wave_uniform(v.x), wave_uniform(v.y), wave_uniform(v.z)};
}

// A workgroup's place among those that share its work: the launch's, or those of its kind
// where one launch advances leptons and photons.
struct Place {
  int block, grid;
};
__device__ __forceinline__ Place launch_place() { return {(int)blockIdx.x, (int)gridDim.x}; }

// Wavefront index among them (wavefront-uniform).
__device__ __forceinline__ int wave_index(Place at) {
  return at.block * (int)(blockDim.x >> 6) +
         __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}
__device__ __forceinline__ int wave_index() { return wave_index(launch_place()); }

// Per-wavefront tally of arena records per instance.  Records are counted for the instance
// `cur` in a register; when another instance shows up the tally goes to the wavefront's own
// word of the count matrix (a private address, so the add never waits on other waves).
struct ArenaTally {
  int cur = -1;
  unsigned n = 0;
  __device__ __forceinline__ void flush(const ChildArena& A, int wid) {
    if (n != 0 && lane_id() == 0)
      atomicAdd(&A.cnt[(size_t)cur * A.waves + wid], n);
    n = 0;
  }
  // Count the flagged lanes (mask m) by instance.  All lanes call it.
  __device__ __forceinline__ void add(const ChildArena& A, int wid, uint64_t m, bool flag,
                                      int inst) {
    while (m) {
      const int leader = __ffsll((unsigned long long)m) - 1;
      const int li = wave_bcast(inst, leader);
      const uint64_t same = wave_ballot(flag && inst == li);
      if (li != cur) {
        flush(A, wid);
        cur = li;
      }
      n += (unsigned)__popcll(same);
      m &= ~same;
    }
  }
};

// A producing wavefront's position in an arena: records written, and the pool chunk it
// fills once its share is full.
struct ArenaCursor {
  long long n = 0;
  unsigned cur = 0xFFFFFFFFu;  // current pool chunk (none yet)
  unsigned fill = (unsigned)kArenaChunk;
};

// Where the ranks of one ballot go: [0, k0) to the share from `share`, [k0, k1) to the
// current chunk from c0, [k1, n) to a new chunk from c1.
struct ArenaSpan {
  long long share, c0, c1;
  int k0, k1;
  __device__ __forceinline__ long long at(int rank) const {
    return rank < k0 ? share + rank : (rank < k1 ? c0 + (rank - k0) : c1 + (rank - k1));
  }
};

// Reserve n_new (1..64) records for one ballot of wavefront wid: the rest of its share,
// then its current chunk, then one new chunk from the pool (one atomic).  False, with
// nothing reserved, when the pool is exhausted.  Wavefront-uniform arguments; all lanes call.
__device__ __forceinline__ bool arena_reserve(const ChildArena& A, int wid, ArenaCursor& c,
                                              int n_new, ArenaSpan& s) {
  const long long room_share = A.per_wave > c.n ? A.per_wave - c.n : 0;
  s.share = (long long)wid * A.per_wave + c.n;
  if (n_new <= room_share) {
    s.k0 = s.k1 = n_new;
    s.c0 = s.c1 = 0;
    c.n += n_new;
    return true;
  }
  s.k0 = (int)room_share;
  const int rest = n_new - s.k0;
  const int room = (int)(kArenaChunk - c.fill);
  s.c0 = A.pool0 + (long long)c.cur * kArenaChunk + c.fill;  // used only if room > 0
  if (rest <= room) {
    s.k1 = n_new;
    s.c1 = 0;
    c.fill += (unsigned)rest;
    c.n += n_new;
    return true;
  }
  unsigned long long nc = 0;
  if (lane_id() == 0) nc = atomicAdd(A.used, 1u);
  nc = (unsigned long long)wave_bcast((long long)nc, 0);
  if (nc >= (unsigned long long)A.nchunks) return false;
  if (lane_id() == 0) {
    if (c.cur == 0xFFFFFFFFu) A.first[wid] = (unsigned)nc;
    else A.next[c.cur] = (unsigned)nc;
  }
  s.k1 = s.k0 + room;
  s.c1 = A.pool0 + (long long)nc * kArenaChunk;
  c.cur = (unsigned)nc;
  c.fill = (unsigned)(rest - room);
  c.n += n_new;
  return true;
}

// The share-only form: false once the ballot does not fit in the rest of the share.
__device__ __forceinline__ bool share_reserve(const ChildArena& A, int wid, ArenaCursor& c,
                                              int n_new, ArenaSpan& s) {
  if (c.n + n_new > A.per_wave) return false;
  s.share = (long long)wid * A.per_wave + c.n;
  s.k0 = s.k1 = n_new;
  s.c0 = s.c1 = 0;
  c.n += n_new;
  return true;
}

// Record indices of producing wavefront sw's records, read in batches [j0, j0 + m) with
// m <= 64 and j0 increasing: advance() (wavefront-uniform) moves to the pool chunk that
// holds the batch's first pool record; index() gives a lane's record j of the batch (below
// n, the wavefront's record count), which lies in the share, that chunk or the next one.
struct ArenaWalk {
  unsigned chunk = 0xFFFFFFFFu;
  long long start = 0;  // the chunk holds pool records [start, start + kArenaChunk) of sw
  __device__ __forceinline__ void advance(const ChildArena& A, int sw, long long j0, long long m,
                                          long long n) {
    if (n <= A.per_wave || j0 + m <= A.per_wave) return;  // the batch is all in the share
    const long long jp = j0 > A.per_wave ? j0 - A.per_wave : 0;
    if (chunk == 0xFFFFFFFFu) {
      chunk = A.first[sw];
      start = 0;
    }
    while (jp >= start + kArenaChunk) {
      chunk = A.next[chunk];
      start += kArenaChunk;
    }
  }
  __device__ __forceinline__ long long index(const ChildArena& A, int sw, long long j) const {
    if (j < A.per_wave) return (long long)sw * A.per_wave + j;
    const long long jp = j - A.per_wave;
    if (jp < start + kArenaChunk) return A.pool0 + (long long)chunk * kArenaChunk + (jp - start);
    return A.pool0 + (long long)A.next[chunk] * kArenaChunk + (jp - start - kArenaChunk);
  }
};

// Current piece of a wavefront's work: slots [cur, end) of one (instance, species) segment.
struct TileCursor {
  long long cur = 0, end = 0;  // slots
  long long g = 0;             // index of slot `cur` in the kernel's particle index space
  int inst = 0, species = 0;
};

// A wavefront's share of the index space [0, N): chunks chunk, chunk + W, ... of T particles.
struct WaveRange {
  long long g, gend, chunk, T, W, N;

  __device__ __forceinline__ void init(Place at, long long n, long long t) {
    W = (long long)at.grid * (blockDim.x >> 6);
    const long long wv = wave_index(at);
    N = n;
    T = t;
    chunk = wv - W;
    g = gend = 0;
  }
  // At particle g of a chunk; false once the wavefront's share is exhausted.
  __device__ __forceinline__ bool more() {
    while (g >= gend) {
      chunk += W;
      const long long s = chunk * T;
      if (s >= N) return false;
      g = s;
      gend = min(s + T, N);
    }
    return true;
  }
  // Next piece within one segment.
  __device__ __forceinline__ bool next(const StepArgs& a, const long long* pref, int nseg,
                                       bool lepton, TileCursor& tc) {
    if (!more()) return false;
    int lo = 0, hi = nseg;  // pref[lo] <= g < pref[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (pref[mid] <= g) lo = mid;
      else hi = mid;
    }
    const int inst = lepton ? (lo >> 1) : lo;
    const int sp = lepton ? (lo & 1) : QED_PHOTON;
    const long long piece_end = min(gend, pref[lo + 1]);
    const long long base = a.inst[inst].base[sp];
    tc.cur = base + (g - pref[lo]);
    tc.end = tc.cur + (piece_end - g);
    tc.g = g;
    tc.inst = inst;
    tc.species = sp;
    g = piece_end;
    return true;
  }
};

// Wavefronts of a kernel of W that own any of N particles in chunks of T (the first ones), and
// workgroups.
__device__ __forceinline__ long long working_waves(long long N, long long W, long long T) {
  // (a 64-bit division costs every workgroup of a launch 0.1 us)
  const int s = T == 128 ? 7 : T == 64 ? 6 : T == 256 ? 8 : T == 512 ? 9 : 0;
  const long long n = s                        ? (N + T - 1) >> s
                      : N < (1ll << 31) - T    ? (long long)(((unsigned)N + (unsigned)T - 1u) / (unsigned)T)
                                               : (N + T - 1) / T;
  return n < W ? n : W;
}
__device__ __forceinline__ int working_blocks(long long N, int grid, int wpb, long long T) {
  return grid > 0 ? (int)((working_waves(N, (long long)grid * wpb, T) + wpb - 1) / wpb) : 0;
}
__device__ __forceinline__ int working_blocks_of(long long N, int grid, int wpb, const Deal& d) {
  return working_blocks(N, grid, wpb, chunk_size(N, (long long)grid * wpb, d));
}
// The chunk of a kind's workgroups, and does this one own any work?
__device__ __forceinline__ long long block_chunk(Place at, long long N, const Deal& d) {
  return chunk_size(N, (long long)at.grid * (blockDim.x >> 6), d);
}
__device__ __forceinline__ bool block_has_work(Place at, long long N, long long T) {
  return at.block < working_blocks(N, at.grid, (int)(blockDim.x >> 6), T);
}

template <bool MIXED>
struct TabType {
  using T = double2;
};
template <>
struct TabType<true> {
  using T = float2;
};

// One draw of the modified generator (Sec. IV.G): r1, r2, delta = r1^3 and
// q = delta / (1 - delta).
struct EmissionDraw {
  double r1, r2, d, q;  // FP64 form
  float f1, f2, fd;     // mixed form
};
template <bool MIXED>
__device__ __forceinline__ EmissionDraw emission_draw(const uint4& o) {
  EmissionDraw e{};
  if (MIXED) {
    e.f1 = uniform32(o.y);
    e.f2 = uniform32(o.w);
    e.fd = e.f1 * e.f1 * e.f1;
  } else {
    e.r1 = uniform64(o.x, o.y);
    e.r2 = uniform64(o.z, o.w);
    e.d = e.r1 * e.r1 * e.r1;
    const double omd = 1.0 - e.d;  // >= 2^-52
    e.q = div_normal(e.d, omd, rcp_normal(omd));
  }
  return e;
}

// Emission decision (Eqs. (24), (25)): emit iff r2 < 3 r1^2 P(r1^3).  The mixed form evaluates
// the rate and the comparison in FP32.  In FP64, with z_scale = (3/2 eps_r)^2, one inverse root
// gives z = (2/3) q / chi = q / sqrt(z_scale c2): at most 4.2 units of 2^-53 from the draw's
// and the state's exact z, where root, products and division had 6 (P takes z times that).
template <bool MIXED>
__device__ __forceinline__ bool emission_decision(const typename TabType<MIXED>::T* tab,
                                                  const MathTab& mt, const Series64& ser64,
                                                  const Series32& ser32, const EmissionDraw& e,
                                                  const Kin& kn, double eps_r, double z_scale,
                                                  double dtfac, LaneCounters& cnt,
                                                  double& delta) {
  if (MIXED) {
    const float chi = (float)(eps_r * root_of(kn.c2).r);
    const float r1 = e.f1, r2 = e.f2;
    const float d = e.fd, omd = 1.0f - d;
    const float z = (2.0f / 3.0f) * d / (omd * chi);
    const float P = 3.0f * r1 * r1 * ((float)(dtfac * kInvSqrt3Pi) / (float)kn.g.r) *
                    emission_bracket32(reinterpret_cast<const float2*>(tab), ser32, z,
                                       d * d / omd);
    cnt.note((double)P, (double)r2);
    delta = (double)d;
    return r2 < P;
  }
  const double d = e.d;
  // a field of 0 is taken as 2^-450 (z_scale infinite: as any): z is beyond the tabulated range
  // and P = 0 either way
  const double w = fmax(z_scale * kn.c2, kFastLo);
  double z = e.q * rsqrt_normal(w);
  double pg = div_normal(dtfac * kInvSqrt3Pi, kn.g.r, kn.g.inv);
  if (!(kn.g.fast && w <= kFastHi)) {
    z = (2.0 / 3.0) * d / ((1.0 - d) * (eps_r * sqrt(kn.c2)));
    pg = kn.g.under(dtfac * kInvSqrt3Pi);
  }
  const double P = 3.0 * e.r1 * e.r1 * pg *
                   emission_bracket64(reinterpret_cast<const double2*>(tab), mt, ser64, z,
                                      d * e.q);
  cnt.note(P, e.r2);
  delta = d;
  return e.r2 < P;
}

// One lane's lepton between its sub-steps: sub-step k, `left` sub-steps of length h to go (the
// current one included).
struct LepLane {
  V3 x{}, p{}, E{}, B{};
  double qh2 = 0.0, h = 0.0, dtfac = 0.0, hs3 = 0.0;
  int k = 0, left = 0;
};

// One sub-step of an active lane: the push, the position and the emission decision for the
// draw o (Sec. IV.G).  A sub-step whose end state breaks Eq. (29) is taken again from its
// start at half the length (rare: such lanes repeat the push while the others wait).
template <bool MIXED, bool HAS_B>
__device__ __forceinline__ bool lepton_substep(const StepArgs& a,
                                               const typename TabType<MIXED>::T* tab,
                                               const MathTab& mt, const Series64& ser64,
                                               const Series32& ser32, uint64_t id, uint64_t seed,
                                               uint32_t step, bool refine, LepLane& L, Kin& kn,
                                               BlockStats& bs, LaneCounters& cnt,
                                               double& delta) {
  const V3 p0 = L.p;
  const bool fast = push_fast<HAS_B>(p0, L.qh2, L.E, L.B, L.p, kn);
  const EmissionDraw e =
      emission_draw<MIXED>(draw_words(id, seed, step, (uint32_t)L.k, kDraw));
  // lhs > rhs: refine; within 4e-12 of each other: the ratio may count as near an integer
  const double rhs = 1.0 + kn.p2;
  if (!fast || (refine && kn.c2 > 0.0 && fma(L.hs3, kn.c2, -rhs) >= -5e-12 * rhs)) {
    if (!fast) push_any<HAS_B>(p0, L.qh2, L.E, L.B, L.p, kn);
    while (refine && kn.c2 > 0.0 &&
           refine_substep(mt, L.hs3, kn, L.h, a.eps_r, a.inv_lep_scale, L.k, L.left, bs)) {
      L.h *= 0.5;
      L.qh2 *= 0.5;
      L.dtfac *= 0.5;
      L.hs3 *= 0.125;
      L.left *= 2;
      push_any<HAS_B>(p0, L.qh2, L.E, L.B, L.p, kn);
    }
  }
  L.x = axpy(kn.g.under(L.h), L.p, L.x);
  if (!a.emission) return false;
  return emission_decision<MIXED>(tab, mt, ser64, ser32, e, kn, a.eps_r, a.z_scale, L.dtfac,
                                  cnt, delta);
}

// The photon of an emission: energy delta gamma m c^2 along p (Sec. IV.F), as the factor
// f = |k| / |p|.  Counts the event's spectrum bin and radiated energy; false (and a
// non-finite count) if p = 0.
__device__ __forceinline__ bool emission_photon(const MathTab& mt, const Kin& kn, double delta,
                                                double wgt, BlockStats& bs, LaneCounters& cnt,
                                                double& f) {
  if (!(kn.p2 > 0.0)) {
    block_count(bs, kPfNonfinite);
    return false;
  }
  const double eps = delta * kn.g.r;
  f = root_of(kn.p2).under(eps);
  // bin floor(10 (log10 eps + 8)), in FP64 in both precisions (an emission is rare next to
  // the sub-steps, and the bins then agree with an FP64 count of the same photons)
  const double s10 = 10.0 * kLog10Of2;
  const double lb = floor(eps >= kFastLo && eps <= kFastHi ? log2_affine(mt, eps, 0, s10, 80.0)
                                                           : fma(log2(eps), s10, 80.0));
  if (lb >= 0.0 && lb < (double)QED_SPECTRUM_BINS) atomicAdd(&bs.w[kPfHist + (int)lb], 1ull);
  cnt.energy += wgt * eps;
  return true;
}

// Same-step processing: the time a child has left in the step and its parent's fields,
// stored with its arena record r (the fields only where they depend on position).
template <int FMODE>
__device__ __forceinline__ void record_same_step(const ChildArena& A, long long r, double tau,
                                                 const V3& E, const V3& B) {
  A.tau[r] = tau;
  if (FMODE == kFieldLocal) {
    const long long c = A.cap;
    double* f = A.fe;
    f[r] = E.x;
    f[c + r] = E.y;
    f[2 * c + r] = E.z;
    f[3 * c + r] = B.x;
    f[4 * c + r] = B.y;
    f[5 * c + r] = B.z;
  }
}

// Column pointer of electrons or positrons without indexing the kernel-argument array.
#define LEPTON_COL(col, sp) ((sp) == QED_ELECTRON ? a.sp[QED_ELECTRON].col : a.sp[QED_POSITRON].col)

// Per-wavefront LDS staging of emitted photons.
struct PhotonStage {
  double x[kStageCap], y[kStageCap], z[kStageCap];
  double px[kStageCap], py[kStageCap], pz[kStageCap], w[kStageCap];
  unsigned long long id[kStageCap], parent[kStageCap];
  unsigned int birth[kStageCap];
  int inst[kStageCap];
};

// Reserve slots for the `staged` records and copy them out (lane j takes record j).
__device__ __forceinline__ void flush_stage(const StepArgs& a, PhotonStage& sg, int staged,
                                            LaneCounters& cnt) {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  const int lane = lane_id();
  const bool has = lane < staged;
  const int j = has ? lane : 0;
  const int rinst = has ? sg.inst[j] : -1;
  wave_append<QED_PHOTON>(a, has, rinst, cnt, [&](const qed_soa& o, long long s) {
    o.x[s] = sg.x[j];
    o.y[s] = sg.y[j];
    o.z[s] = sg.z[j];
    o.px[s] = sg.px[j];
    o.py[s] = sg.py[j];
    o.pz[s] = sg.pz[j];
    o.w[s] = sg.w[j];
    o.id[s] = sg.id[j];
    o.parent[s] = sg.parent[j];
    o.birth[s] = sg.birth[j];
    if (o.n_events) o.n_events[s] = 0u;
  });
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// Per-wavefront LDS staging of pair creations (one record -> an electron and a positron).
struct PairStage {
  double x[kStageCap], y[kStageCap], z[kStageCap];
  double kx[kStageCap], ky[kStageCap], kz[kStageCap], r1[kStageCap], w[kStageCap];
  unsigned long long parent[kStageCap];
  unsigned int sub[kStageCap];
  int inst[kStageCap];
};

__device__ __forceinline__ void flush_pairs(const StepArgs& a, PairStage& sg, int staged,
                                            uint32_t step, LaneCounters& cnt) {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  const int lane = lane_id();
  const bool has = lane < staged;
  const int j = has ? lane : 0;
  const int rinst = has ? sg.inst[j] : -1;
  const uint64_t seed = has ? a.inst[rinst].seed : 0ull;
  const double r1 = sg.r1[j];
  // electron takes r1 of the photon momentum, positron the rest (Sec. V.A)
  wave_append<QED_ELECTRON>(a, has, rinst, cnt, [&](const qed_soa& o, long long s) {
    o.x[s] = sg.x[j];
    o.y[s] = sg.y[j];
    o.z[s] = sg.z[j];
    o.px[s] = r1 * sg.kx[j];
    o.py[s] = r1 * sg.ky[j];
    o.pz[s] = r1 * sg.kz[j];
    o.w[s] = sg.w[j];
    o.id[s] = child_id(sg.parent[j], seed, step, sg.sub[j], kElectronChild);
    o.parent[s] = sg.parent[j];
    o.birth[s] = birth_code(step, sg.sub[j]);
    if (o.n_events) o.n_events[s] = 0u;
  });
  wave_append<QED_POSITRON>(a, has, rinst, cnt, [&](const qed_soa& o, long long s) {
    const double r1c = 1.0 - r1;
    o.x[s] = sg.x[j];
    o.y[s] = sg.y[j];
    o.z[s] = sg.z[j];
    o.px[s] = r1c * sg.kx[j];
    o.py[s] = r1c * sg.ky[j];
    o.pz[s] = r1c * sg.kz[j];
    o.w[s] = sg.w[j];
    o.id[s] = child_id(sg.parent[j], seed, step, sg.sub[j], kPositronChild);
    o.parent[s] = sg.parent[j];
    o.birth[s] = birth_code(step, sg.sub[j]);
    if (o.n_events) o.n_events[s] = 0u;
  });
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// ------------------------------------------------------------------------------------
// leptons
// ------------------------------------------------------------------------------------
// EXT: the extensions are compiled in -- the generator factor, and same-step processing
// (children also get their time left and the parent's fields; a full share continues in
// pool chunks).  Without them a full share falls back to direct reservation, and the plain
// step's kernel stays lean.
//
// The emission table goes to LDS (64 KB in FP64, 32 KB in FP32), except in the plain FP64
// kernel for a space-independent E with B = 0: there it is read from the L2-resident copy,
// and without the 64 KB of LDS per workgroup the kernel fits three wavefronts per SIMD (the
// compiler holds it to 168 VGPRs with a few spilled), 8% faster on the rotating-field
// cascade.  With a B field the Boris rotation's registers make that bound cost more spills
// than the third wavefront gains (3% slower on 10^4 electrons in a uniform B), and with a
// grid field far more (1.9 times slower), so those kernels keep the LDS table at two
// wavefronts per SIMD.  The mixed form's table is half as large, and three workgroups' LDS fits a
// CU: its kernels for space-independent fields are held to three wavefronts as well (with a B
// field 17 registers spill; two against three wavefronts, us a step of 10^6 leptons and 10^3
// photons: rotating 109 / 94, uniform B 123 / 113; with 10^6 photons 138 / 120, 152 / 136; leptons
// alone 102 / 91, 119 / 110).  The extended forms get two at least, one in a
// position-dependent field needs 256 VGPRs and spills a few.
template <bool MIXED, int FMODE, bool EXT>
struct LeptonShape {
  static constexpr bool global_table = !MIXED && FMODE == kFieldE && !EXT;
  static constexpr int min_waves =
      global_table || (MIXED && FMODE != kFieldLocal && !EXT) ? 3 : EXT ? 2 : 1;
};

// The lepton kernels' LDS.
template <bool MIXED, int FMODE, bool EXT>
struct LeptonLds {
  typename TabType<MIXED>::T tab[LeptonShape<MIXED, FMODE, EXT>::global_table ? 1 : kTableN];
  BlockStats bs;
  MathTab mt;
  PhotonStage stage[kWavesPerBlock];
};

// RUNS: the reverse mode of Sec. VI (runs_photon > 1) is compiled in (with EXT).
template <bool MIXED, int FMODE, bool EXT, bool RUNS>
__device__ __forceinline__ void lepton_step(const StepArgs& a, Place at,
                                            LeptonLds<MIXED, FMODE, EXT>& lds) {
  using Tab = typename TabType<MIXED>::T;
  constexpr bool kGlobalTab = LeptonShape<MIXED, FMODE, EXT>::global_table;
  BlockStats& bs = lds.bs;
  MathTab& mt = lds.mt;
  const MathRow mrow = load_math();
  WorkHdr* hdr = a.hdr;
  const long long N = hdr->lep_total;
  const int wid = wave_index(at);
  const long long chunk = block_chunk(at, N, a.lep_deal);
  if (!block_has_work(at, N, chunk)) {
    if (a.pa.waves > 0 && lane_id() == 0) a.pa.nrec[wid] = 0u;
    return;
  }
  block_stats_init(bs);
  const Tab* src = MIXED ? reinterpret_cast<const Tab*>(a.tables->ab32)
                         : reinterpret_cast<const Tab*>(a.tables->ab64);
  if (!kGlobalTab)
    for (int i = threadIdx.x; i < kTableN; i += blockDim.x) lds.tab[i] = src[i];
  const Tab* tab = kGlobalTab ? src : lds.tab;
  store_math(mt, mrow);
  __syncthreads();

  const Series64 ser64 = {a.tables->series[0], a.tables->series[1], a.tables->series[2],
                          a.tables->series[3], a.tables->series[4]};
  const Series32 ser32 = {(float)ser64.b0, (float)ser64.b1, (float)ser64.c0, (float)ser64.c1,
                          (float)ser64.c2};
  const uint32_t step = (uint32_t)hdr->step;
  const int nseg = 2 * a.n_inst;
  FieldArgs fld = a.field;
  fld.tn = hdr->tn;
  const uint64_t below = lanes_below();
  PhotonStage& sg = lds.stage[threadIdx.x >> 6];

  LaneCounters cnt;
  cnt.bs = &bs;
  WaveCounters wc;
  TileCursor tc;
  WaveRange wr;
  wr.init(at, N, chunk);
  bool open = true;
  int staged = 0;
  // arena: this wavefront's share, then pool chunks
  const ChildArena& pa = a.pa;
  ArenaCursor acur;
  ArenaTally tally;

  // lane state: the particle in `slot`
  long long slot = -1;
  int inst = 0, sp = 0;
  LepLane L;
  V3 &x = L.x, &p = L.p, &E = L.E, &B = L.B;
  int &k = L.k, &left = L.left;
  double &h = L.h;
  uint64_t id = 0, seed = 0;
  uint32_t nev = 0;
  double wgt = 0.0;
  const bool refine = a.forced <= 0 && a.adaptive;

  while (true) {
    // ---- refill idle lanes from the wavefront's share, once enough of them are idle ----
    uint64_t freem = wave_ballot(slot < 0);
    if (__popcll(freem) < a.refill_min && ~freem != 0ull) freem = 0ull;
    while (freem != 0 && open) {
      if (tc.cur >= tc.end) {
        open = wr.next(a, a.lep_pref, nseg, true, tc);
        continue;
      }
      const int nfree = __popcll(freem);
      const long long avail = tc.end - tc.cur;
      const int take = (int)(avail < nfree ? avail : nfree);
      const int rank = __popcll(freem & below);
      if (slot < 0 && rank < take) {
        slot = tc.cur + rank;
        inst = tc.inst;
        sp = tc.species;
        x = {LEPTON_COL(x, sp)[slot], LEPTON_COL(y, sp)[slot], LEPTON_COL(z, sp)[slot]};
        p = {LEPTON_COL(px, sp)[slot], LEPTON_COL(py, sp)[slot], LEPTON_COL(pz, sp)[slot]};
        id = LEPTON_COL(id, sp)[slot];
        wgt = LEPTON_COL(w, sp)[slot];
        uint32_t* ne = LEPTON_COL(n_events, sp);
        nev = ne ? ne[slot] : 0u;
        seed = a.inst[inst].seed;
        if (FMODE == kFieldLocal) {
          field_at_position(fld, a.inst[inst].amp, x, E, B);
        } else {
          const double* eb = a.eb + 6 * inst;
          E = {eb[0], eb[1], eb[2]};
          if (FMODE == kFieldEB) B = {eb[3], eb[4], eb[5]};
        }
        // chi and the number of sub-steps, once per step from the step-start state
        const Kin kn = kin_of<FMODE != kFieldE>(p, E, B);
        // (FP64 in both precisions: n_sub is no part of the FP32 rate evaluation)
        int nsub = 1;
        if (a.forced > 0) {
          nsub = a.forced;
        } else if (a.adaptive && kn.c2 > 0.0) {
          const NsubInfo ni =
              nsub_from_ratio(substep_ratio_lepton(mt, a.dt, kn, a.eps_r, a.inv_lep_scale));
          nsub = ni.n;
          if (ni.near_int) block_count(bs, kPfNearInt);
          if (ni.clamped) block_count(bs, kPfClamped);
        }
        if (!isfinite(kn.c2)) block_count(bs, kPfNonfinite);
        atomicAdd(&bs.w[kPfNsub + (nsub < QED_NSUB_HIST ? nsub : QED_NSUB_HIST - 1)], 1ull);
        h = div_normal(a.dt, (double)nsub, rcp_normal((double)nsub));
        L.dtfac = h * a.dtfac_per_h;
        L.qh2 = (sp == QED_ELECTRON ? -0.5 : 0.5) * h;
        L.hs3 = a.eps_r * a.eps_r * substep_cube(h, a.inv_lep_scale);
        k = 0;
        left = nsub;
      }
      if (tc.species == QED_ELECTRON) wc.adv0 += take;
      else wc.adv1 += take;
      tc.cur += take;
      freem = wave_ballot(slot < 0);
    }
    const uint64_t act = wave_ballot(slot >= 0);
    if (act == 0) break;

    // ---- one sub-step: push, chi, emission decision (Sec. IV.G) ----
    bool emit = false;
    double f = 0.0;
    Kin kn{0.0, 0.0, {1.0, 1.0, true}};
    // the weight of an event's photon before any factor: w, or w / N_g in the reverse mode
    // of Sec. VI, whose runs beyond the first follow the first below
    const double wrun = RUNS ? wgt / (double)a.runs_photon : wgt;
    // With same-step children (large steps: few leptons, hundreds of sub-steps) sub-steps follow
    // each other here until a lane emits or ends its last one; nothing below concerns the others,
    // and its tests took a fifth of each sub-step (with the same in the generation kernel:
    // shower 17.1 to 14.5 ms, avalanche 35.6 to 30.5).  The plain kernels emit in nearly every
    // sub-step of a full wavefront, and the loop's registers cost them more than it saves
    // (rotating cascade 138 to 152 ms, grid cascade 35.4 to 40.9).
    int iters = 0;
    for (;;) {
      ++iters;
      if (slot >= 0) {
        double delta;
        if (lepton_substep<MIXED, FMODE != kFieldE>(a, tab, mt, ser64, ser32, id, seed, step,
                                                    refine, L, kn, bs, cnt, delta)) {
          emit = emission_photon(mt, kn, delta, wrun, bs, cnt, f);
          if (emit) ++nev;
        }
      }
      if (!EXT || RUNS || wave_ballot(slot >= 0 && (emit || left == 1))) break;
      ++k;
      --left;
    }
    wc.wave_iters += iters;
    wc.low_occ += __popcll(act) < 32 ? iters : 0;
    wc.substeps += (long long)iters * __popcll(act);

    // ---- emitted photons: into the wavefront's arena share, else staged and reserved ----
    // With a generator factor f_g (Sec. VI) the photon of an event is created with
    // probability 1 / f_g, or for every f_g-th event of the lepton in the deterministic
    // form, and carries f_g times the lepton's weight; the recoil below happens at every
    // event.
    bool child = emit;
    if (EXT && emit) {
      if (a.every_photon) child = generator_every(id, seed, nev - 1u, a.every_photon);
      else if (a.fg_photon > 1.0)
        child = generator_runs(id, seed, step, (uint32_t)k, kGenPhoton, a.inv_fg_photon);
    }
    const double cw = RUNS ? wrun : EXT ? wgt * a.fg_photon : wgt;
    const bool ss = EXT && a.generations > 0;
    const uint64_t em = wave_ballot(child);
    ArenaSpan span;
    if (em && pa.waves > 0 &&
        (EXT ? arena_reserve(pa, wid, acur, __popcll(em), span)
             : share_reserve(pa, wid, acur, __popcll(em), span))) {
      const int n_new = __popcll(em);
      wc.events += n_new;
      tally.add(pa, wid, em, child, inst);
      if (child) {
        const long long r = span.at(__popcll(em & below));
        pa.x[r] = x.x;
        pa.y[r] = x.y;
        pa.z[r] = x.z;
        pa.px[r] = f * p.x;
        pa.py[r] = f * p.y;
        pa.pz[r] = f * p.z;
        pa.w[r] = cw;
        pa.parent[r] = id;
        pa.sub[r] = (unsigned)k;
        pa.inst[r] = (unsigned)inst;
        if (ss) record_same_step<FMODE>(pa, r, (double)(left - 1) * h, E, B);
      }
    } else if (em) {
      const int n_new = __popcll(em);
      wc.events += n_new;
      // reserved directly in the stores: not advanced in this step
      if (ss) wc.deferred += __popcll(wave_ballot(child && left > 1));
      if (staged + n_new > kStageCap) {
        flush_stage(a, sg, staged, cnt);
        staged = 0;
      }
      if (n_new > kStageCap) {
        wave_append<QED_PHOTON>(a, child, inst, cnt, [&](const qed_soa& o, long long s) {
          o.x[s] = x.x;
          o.y[s] = x.y;
          o.z[s] = x.z;
          o.px[s] = f * p.x;
          o.py[s] = f * p.y;
          o.pz[s] = f * p.z;
          o.w[s] = cw;
          o.id[s] = child_id(id, seed, step, (uint32_t)k, kPhotonChild);
          o.parent[s] = id;
          o.birth[s] = birth_code(step, (uint32_t)k);
          if (o.n_events) o.n_events[s] = 0u;
        });
      } else {
        if (child) {
          const int r = staged + __popcll(em & below);
          sg.x[r] = x.x;
          sg.y[r] = x.y;
          sg.z[r] = x.z;
          sg.px[r] = f * p.x;
          sg.py[r] = f * p.y;
          sg.pz[r] = f * p.z;
          sg.w[r] = cw;
          sg.id[r] = child_id(id, seed, step, (uint32_t)k, kPhotonChild);
          sg.parent[r] = id;
          sg.birth[r] = birth_code(step, (uint32_t)k);
          sg.inst[r] = inst;
        }
        staged += n_new;
      }
    }
    if constexpr (RUNS) {
      // reverse mode: runs 1 .. N_g - 1 of the generator on the same state, each photon
      // appended as above; the lepton then recoils by the mean of the runs' photons
      V3 rec = {0.0, 0.0, 0.0};
      if (emit) rec = {f * p.x, f * p.y, f * p.z};
      bool fired = emit;
      for (int run = 1; run < a.runs_photon; ++run) {
        const uint32_t sc = sub_code(k, run);
        bool e2 = false;
        double f2 = 0.0;
        if (slot >= 0 && a.emission) {
          const uint4 o = draw_words(id, seed, step, sc, kDraw);
          double delta;
          e2 = emission_decision<MIXED>(tab, mt, ser64, ser32, emission_draw<MIXED>(o), kn,
                                        a.eps_r, a.z_scale, L.dtfac, cnt, delta);
          if (e2) {
            e2 = emission_photon(mt, kn, delta, wrun, bs, cnt, f2);
            if (e2) ++nev;
          }
        }
        const uint64_t em2 = wave_ballot(e2);
        if (em2) {
          const int n_new = __popcll(em2);
          wc.events += n_new;
          ArenaSpan span2;
          if (pa.waves > 0 && arena_reserve(pa, wid, acur, n_new, span2)) {
            tally.add(pa, wid, em2, e2, inst);
            if (e2) {
              const long long r = span2.at(__popcll(em2 & below));
              pa.x[r] = x.x;
              pa.y[r] = x.y;
              pa.z[r] = x.z;
              pa.px[r] = f2 * p.x;
              pa.py[r] = f2 * p.y;
              pa.pz[r] = f2 * p.z;
              pa.w[r] = wrun;
              pa.parent[r] = id;
              pa.sub[r] = sc;
              pa.inst[r] = (unsigned)inst;
              if (ss) record_same_step<FMODE>(pa, r, (double)(left - 1) * h, E, B);
            }
          } else {
            // reserved directly in the stores: not advanced in this step
            if (ss) wc.deferred += __popcll(wave_ballot(e2 && left > 1));
            wave_append<QED_PHOTON>(a, e2, inst, cnt, [&](const qed_soa& o, long long s) {
              o.x[s] = x.x;
              o.y[s] = x.y;
              o.z[s] = x.z;
              o.px[s] = f2 * p.x;
              o.py[s] = f2 * p.y;
              o.pz[s] = f2 * p.z;
              o.w[s] = wrun;
              o.id[s] = child_id(id, seed, step, sc, kPhotonChild);
              o.parent[s] = id;
              o.birth[s] = birth_code(step, (uint32_t)k);
              if (o.n_events) o.n_events[s] = 0u;
            });
          }
        }
        if (e2) {
          rec = {rec.x + f2 * p.x, rec.y + f2 * p.y, rec.z + f2 * p.z};
          fired = true;
        }
      }
      if (fired) {
        const double R = (double)a.runs_photon;
        p = {p.x - rec.x / R, p.y - rec.y / R, p.z - rec.z / R};
      }
      emit = false;  // the recoil is done
    }
    if (emit) {
      // recoil: the lepton keeps p - k (momentum conservation, Sec. IV.F)
      p = recoil(p, f);
    }

    // ---- lanes whose particle has done all its sub-steps write back and go idle ----
    if (slot >= 0 && (++k, --left == 0)) {
      LEPTON_COL(x, sp)[slot] = x.x;
      LEPTON_COL(y, sp)[slot] = x.y;
      LEPTON_COL(z, sp)[slot] = x.z;
      LEPTON_COL(px, sp)[slot] = p.x;
      LEPTON_COL(py, sp)[slot] = p.y;
      LEPTON_COL(pz, sp)[slot] = p.z;
      uint32_t* ne = LEPTON_COL(n_events, sp);
      if (ne) ne[slot] = nev;
      slot = -1;
    }
  }
  if (staged > 0) flush_stage(a, sg, staged, cnt);
  if (pa.waves > 0) {
    tally.flush(pa, wid);
    if (lane_id() == 0) pa.nrec[wid] = (unsigned)acur.n;
  }

  wave_to_block(bs, cnt, wc);
  __syncthreads();
  block_stats_store(bs, a.lep_part, kPfCount, at.block);
}

template <bool MIXED, int FMODE, bool EXT>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(LeptonShape<MIXED, FMODE, EXT>::min_waves)))
    lepton_kernel(StepArgs a) {
  __shared__ LeptonLds<MIXED, FMODE, EXT> lds;
  lepton_step<MIXED, FMODE, EXT, false>(a, launch_place(), lds);
}

// The reverse mode of Sec. VI in a kernel of its own: its extra runs hold more registers,
// which the other forms would pay for in occupancy.  Held to two wavefronts per SIMD (a few
// spilled registers) rather than one.
template <bool MIXED, int FMODE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
    lepton_runs_kernel(StepArgs a) {
  __shared__ LeptonLds<MIXED, FMODE, true> lds;
  lepton_step<MIXED, FMODE, true, true>(a, launch_place(), lds);
}

// ------------------------------------------------------------------------------------
// photons
// ------------------------------------------------------------------------------------
// Photons keep chi_gamma fixed over the step (fields frozen, k unchanged), almost always
// need a single sub-step, and are mostly far from pair threshold: a per-octave bound of
// the pair probability settles those decisions from r2 alone.  Two kernels:
//   photon_kernel -- each lane takes the next photon of the wavefront's chunk: fields,
//             chi_gamma, n_sub, then for each sub-step the push and the draw; a draw with
//             r2 below the bound makes the photon a candidate -- its index and sub-step go
//             to a list in the workspace -- and its processing stops there;
//   photon_exact_kernel -- each lane re-derives one candidate's state from the stores (same
//             arithmetic, same draws), evaluates the pair probability of Eq. (30) at the
//             recorded sub-step, finishes the photon's sub-steps and stages the pairs.
// The table lookups, logarithms and exponentials stay out of the bulk kernel, whose small
// register footprint lets many wavefronts stay resident to hide HBM latency.

struct PhotonSetup {
  double chi, h, hk, pref, pbound;
  int nsub;
};

// chi_gamma, n_sub and the rate prefactors of one photon in the fields E, B (identical in
// both photon kernels).  `bound` holds the per-octave pair-rate bounds (staged in LDS).
template <bool MIXED, bool HAS_B>
__device__ __forceinline__ PhotonSetup photon_setup(const StepArgs& a, const V3& E, const V3& B,
                                                    const V3& kv, double kabs, double inv_k,
                                                    const double* bound, BlockStats* bs) {
  PhotonSetup ps;
  // chi_gamma (Eqs. (31), (32))
  ps.chi = a.eps_r * root_of(chi_sq<HAS_B>(kv, kabs, E, B)).r;
  ps.nsub = 1;
  if (a.forced > 0) {
    ps.nsub = a.forced;
  } else if (a.adaptive && ps.chi > 0.0) {
    // dt / dt_q with dt_q = kappa 130 (2 pi eps_r) |k| / chi_gamma (Eq. (33))
    const NsubInfo ni = nsub_from_ratio(a.dt * (ps.chi * inv_k) * a.inv_pho_scale);
    ps.nsub = ni.n;
    if (bs) {
      if (ni.near_int) block_count(*bs, kPfNearInt);
      if (ni.clamped) block_count(*bs, kPfClamped);
    }
  }
  if (bs && !isfinite(ps.chi)) block_count(*bs, kPfNonfinite);
  const double h = ps.nsub == 1 ? a.dt : div_normal(a.dt, (double)ps.nsub, rcp_normal((double)ps.nsub));
  ps.h = h;
  ps.hk = h * inv_k;
  ps.pref = h * (a.dtfac_per_h * kInvSqrt3Pi) * inv_k;
  // upper bound of the pair probability over delta_e for this chi's sub-octave
  ps.pbound = 0.0;
  if (ps.chi > 0.0) {
    int e2;
    const double m = frexp(ps.chi, &e2);  // chi = m 2^e2, m in [1/2, 1)
    const int oi = e2 + kBoundOffset;
    if (oi >= kBoundOctaves) {
      ps.pbound = __builtin_inf();
    } else if (oi >= 0) {
      int j = (int)((2.0 * m - 1.0) * kBoundSub);  // exact: chi < (1/2 + (j+1)/32) 2^e2
      j = j < kBoundSub - 1 ? j : kBoundSub - 1;
      ps.pbound = ps.pref * bound[oi * kBoundSub + j];
    }
  }
  return ps;
}

// The per-octave pair-rate bounds into LDS (FP32 values widened in the mixed form).
template <bool MIXED>
__device__ __forceinline__ void stage_bounds(const StepArgs& a, double* sb) {
  for (int i = threadIdx.x; i < kBoundEntries; i += blockDim.x)
    sb[i] = MIXED ? (double)a.tables->pair_bound32[i] : a.tables->pair_bound64[i];
}

// Space-independent fields of a (wavefront-uniform) instance.
template <int FMODE>
__device__ __forceinline__ void instance_fields(const StepArgs& a, int inst, V3& E, V3& B) {
  const double* eb = a.eb + 6 * inst;
  E = {eb[0], eb[1], eb[2]};
  B = FMODE == kFieldEB ? V3{eb[3], eb[4], eb[5]} : V3{0.0, 0.0, 0.0};
}

// Can a draw fall below the bound at all?  The smallest uniform is 2^-53 in FP64 and 2^-24
// in FP32, so a smaller bound settles the decision without drawing.
template <bool MIXED>
__device__ __forceinline__ bool bound_reachable(double pbound) {
  if (MIXED) return (float)pbound > 0x1p-24f;
  return pbound > 0x1p-53;
}

// Below the bound?  (the mixed path compares in FP32, as its exact evaluation does)
template <bool MIXED>
__device__ __forceinline__ bool below_bound(const uint4& o, double pbound) {
  if (MIXED) return uniform32(o.w) < (float)pbound;
  return uniform64(o.z, o.w) < pbound;
}

// Exact pair decision of Eq. (30) for draw o; returns r1 through *r1out.
template <bool MIXED>
__device__ __forceinline__ bool pair_decision(const StepArgs& a, const MathTab& mt,
                                              const Series64& s64, const Series32& s32, const uint4& o, double chi,
                                              double pref, LaneCounters& cnt, double* r1out) {
  if (MIXED) {
    const float r1 = uniform32(o.y), r2 = uniform32(o.w);
    const float omd = 1.0f - r1;
    const float z = (2.0f / 3.0f) / ((float)chi * r1 * omd);
    const float P = (float)pref * pair_bracket32(a.tables->bc32, s32, z, r1 / omd + omd / r1);
    cnt.note((double)P, (double)r2, r2 < P);
    *r1out = (double)r1;
    return r2 < P;
  }
  const double r1 = uniform64(o.x, o.y), r2 = uniform64(o.z, o.w);
  const double omd = 1.0 - r1;  // r1 and 1 - r1 >= 2^-53
  const double z = (2.0 / 3.0) / (chi * r1 * omd);
  const double cB = div_normal(r1, omd, rcp_normal(omd)) + div_normal(omd, r1, rcp_normal(r1));
  const double P = pref * pair_bracket64(a.tables->bc64, mt, s64, z, cB);
  cnt.note(P, r2, r2 < P);
  *r1out = r1;
  return r2 < P;
}

// Columns of the n <= 64 photon slots from `base` on for one wavefront (lane i takes base + i,
// the lanes from n on the last one's again).  `base` is wavefront-uniform, so every column is
// addressed by one scalar base and a lane offset.
struct PhotonIn {
  uint64_t id;
  V3 x, k;
};
__device__ __forceinline__ PhotonIn load_photons(const qed_soa& S, long long base, int n,
                                                 int lane) {
  PhotonIn r;
  const int i = min(lane, n - 1);
  // the columns this kernel only reads are streamed past the caches (non-temporal): 3%
  // faster; the positions, which it writes back, are slower read that way
  r.id = __builtin_nontemporal_load(&S.id[base + i]);
  r.x = {S.x[base + i], S.y[base + i], S.z[base + i]};
  r.k = {__builtin_nontemporal_load(&S.px[base + i]), __builtin_nontemporal_load(&S.py[base + i]),
         __builtin_nontemporal_load(&S.pz[base + i])};
  return r;
}

struct PhotonLds {
  BlockStats bs;
  double bound[kBoundEntries];
};

// One batch of a photon wavefront: the n slots from `base` on, requested but not waited for
// (n = 0: the wavefront has no more).
struct PhotonBatch {
  PhotonIn in;
  long long base = 0, g = 0;  // slot and index in the kernel's particle index space
  int n = 0, inst = 0;
};
// A photon wavefront's batches in turn.  Loads come back in their order, and the compiler waits
// for as many as the path with the fewest has issued: so every fetch issues its loads, the ones
// past the end those of the last batch again (or of slot 0), and an instance's segment is looked
// up once for all the pieces in it.
struct PhotonStream {
  WaveRange wr;
  long long pos = 0, end = 0;      // slots of the current piece
  long long seg_end = 0, off = 0;  // end of the current segment, slot - index in it
  long long last = 0;              // first slot of the last batch
  int inst = 0;
  __device__ __forceinline__ void fetch(const StepArgs& a, const qed_soa& S, int lane,
                                        PhotonBatch& b) {
    if (pos >= end && wr.more()) {
      if (wr.g >= seg_end) {
        int lo = 0, hi = a.n_inst;  // pho_pref[lo] <= g < pho_pref[hi]
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (wave_uniform(a.pho_pref[mid]) <= wr.g) lo = mid;
          else hi = mid;
        }
        inst = lo;
        seg_end = wave_uniform(a.pho_pref[lo + 1]);
        off = wave_uniform(a.inst[lo].base[QED_PHOTON] - a.pho_pref[lo]);
      }
      pos = wr.g + off;
      wr.g = min(wr.gend, seg_end);
      end = wr.g + off;
    }
    b.n = (int)min(end - pos, 64ll);
    if (b.n > 0) last = pos;
    b.base = last;
    b.g = last - off;
    b.inst = inst;
    // the loads go out at a raised wave priority, ahead of the other wavefronts' arithmetic on
    // the SIMD (265 against 267 us per launch on the rotating-field cascade)
    __builtin_amdgcn_s_setprio(1);
    b.in = load_photons(S, last, max(b.n, 1), lane);
    __builtin_amdgcn_s_setprio(0);
    pos += b.n;
  }
};

template <bool MIXED, int FMODE, int DEPTH>
__device__ __forceinline__ void photon_step(const StepArgs& a, Place at, PhotonLds& lds) {
  BlockStats& bs = lds.bs;
  double* const sbound = lds.bound;
  WorkHdr* hdr = a.hdr;
  const long long N = hdr->pho_total;
  const int wid = wave_index(at);
  const long long chunk = block_chunk(at, N, a.pho_deal);
  if (!block_has_work(at, N, chunk)) return;
  block_stats_init(bs);
  stage_bounds<MIXED>(a, sbound);
  __syncthreads();
  const uint32_t step = (uint32_t)hdr->step;
  FieldArgs fld = a.field;
  fld.tn = hdr->tn;
  const uint64_t below = lanes_below();
  const int lane = lane_id();
  const qed_soa& S = a.sp[QED_PHOTON];
  // this wavefront's candidate list; a full list spills to the shared overflow list
  unsigned long long* clist = a.candw + (size_t)wid * a.cand_per_wave;
  long long ncand = 0;

  LaneCounters cnt;
  cnt.bs = &bs;
  WaveCounters wc;
  PhotonStream st;
  st.wr.init(at, N, chunk);

  // Software pipeline: DEPTH batches of 64 photons are requested before the current one is
  // processed, so each wavefront keeps loads in flight while it computes.  One in a launch of
  // its own (four wavefronts per SIMD and more), two beside the leptons, whose registers and LDS
  // leave three wavefronts per SIMD or two.  With one batch, and look-ups in between that
  // waited for all loads, a step of 2 10^5 leptons and 1.6 10^7 photons took 361 us in the
  // rotating field and 423 in a uniform B (FP64), against 346 and 357 in a launch each; with
  // two 335 and 345.
  int inst = -1;
  uint64_t seed = 0;
  double amp = 0.0;
  V3 Ei{}, Bi{};
  auto process = [&](const PhotonIn& in, long long base, long long g0, int n) {
    V3 E = Ei, B = Bi;
    double* X = S.x + base;
    double* Y = S.y + base;
    double* Z = S.z + base;
    bool cand = false;
    int kcand = 0;
    const uint64_t id = in.id;
    V3 x = in.x;
    const V3 kv = in.k;
    const Root kr = root_of(dot(kv, kv));
    const double kabs = kr.r, inv_k = kr.under(1.0);
    const bool live = lane < n && id != QED_ID_DEAD;
    const bool ok = live && kabs > 0.0 && isfinite(kabs);
    if (live && !ok) block_count(bs, kPfNonfinite);
    wc.adv0 += __popcll(wave_ballot(ok));
    if (ok) {
      if (FMODE == kFieldLocal) field_at_position<true>(fld, amp, x, E, B);
      const PhotonSetup ps = photon_setup<MIXED, FMODE != kFieldE>(a, E, B, kv, kabs, inv_k,
                                                                   sbound, &bs);
      int k = 0;
      for (; k < ps.nsub; ++k) {
        if (a.push_photons) x = {x.x + ps.hk * kv.x, x.y + ps.hk * kv.y, x.z + ps.hk * kv.z};
        if (!a.pairs) continue;
        if (!bound_reachable<MIXED>(ps.pbound)) {
          cnt.early += a.runs_pair;
          continue;
        }
        // a candidate if the draw of any run (N_g of them in the reverse mode of Sec. VI)
        // falls below the bound
        bool hit = below_bound<MIXED>(draw_words(id, seed, step, (uint32_t)k, kDraw),
                                      ps.pbound);
        for (int run = 1; run < a.runs_pair && !hit; ++run)
          hit = below_bound<MIXED>(draw_words(id, seed, step, sub_code(k, run), kDraw),
                                   ps.pbound);
        if (hit) {
          cand = true;
          kcand = k;
          break;
        }
        cnt.early += a.runs_pair;
      }
      if (!cand) {
        cnt.subs += ps.nsub;
        if (a.push_photons) {
          // streaming stores: the positions are not read again in this step (1% faster
          // than plain stores; reading the positions non-temporally as well was slower)
          __builtin_nontemporal_store(x.x, &X[lane]);
          __builtin_nontemporal_store(x.y, &Y[lane]);
          __builtin_nontemporal_store(x.z, &Z[lane]);
        }
      } else {
        cnt.subs += kcand;  // the exact kernel counts the rest
      }
    }
    // ---- record candidates: (photon index << 16) | sub-step ----
    const uint64_t cm = wave_ballot(cand);
    if (cm) {
      const int nc = __popcll(cm);
      const unsigned long long e =
          ((unsigned long long)(g0 + lane) << 16) | (unsigned long long)kcand;
      if (ncand + nc <= a.cand_per_wave) {
        if (cand) clist[ncand + __popcll(cm & below)] = e;
        ncand += nc;
      } else {
        unsigned long long pos = 0;
        if (lane == 0) pos = atomicAdd(&hdr->n_cand, (unsigned long long)nc);
        pos = (unsigned long long)wave_bcast((long long)pos, 0) + (unsigned long long)__popcll(cm & below);
        // the overflow list holds one entry per photon slot: never full
        if (cand && pos < (unsigned long long)a.cand_cap) a.cand[pos] = e;
      }
    }
  };
  auto turn = [&](PhotonBatch& b) {
    if (b.inst != inst) {
      inst = b.inst;
      seed = (uint64_t)wave_uniform((long long)a.inst[inst].seed);
      if (FMODE == kFieldLocal) {
        amp = wave_uniform(a.inst[inst].amp);
      } else {
        instance_fields<FMODE>(a, inst, Ei, Bi);
        Ei = wave_uniform(Ei);
        Bi = wave_uniform(Bi);
      }
    }
    const PhotonIn in = b.in;
    const long long base = b.base, g0 = b.g;
    const int n = b.n;
    st.fetch(a, S, lane, b);
    process(in, base, g0, n);
  };
  PhotonBatch b0, b1;
  st.fetch(a, S, lane, b0);
  if (DEPTH > 1) st.fetch(a, S, lane, b1);
  while (b0.n > 0) {
    turn(b0);
    if (DEPTH > 1) {
      if (b1.n <= 0) break;
      turn(b1);
    }
  }
  if (lane == 0) a.candn[wid] = (unsigned)ncand;
  wave_to_block(bs, cnt, wc);
  __syncthreads();
  block_stats_store(bs, a.pho_part, kPfNsub, at.block);
}

template <bool MIXED, int FMODE>
__global__ void __launch_bounds__(256) photon_kernel(StepArgs a) {
  __shared__ PhotonLds lds;
  photon_step<MIXED, FMODE, 1>(a, launch_place(), lds);
}

// Leptons and photons of a step in one launch (no same-step children): neither reads what the
// other writes.  The leptons' arithmetic and the photons' memory traffic share the CUs, the tail
// of one is filled by the other, and a launch is saved.  The workgroups go out in groups of one
// per CU (a multiple of the XCDs, so that a workgroup's XCD stays its index modulo 8): the
// leptons first (lepton_blocks), then the photons into the places they leave.  Where the photons
// are most of the work (kInterleave times the leptons or more), one group of leptons and as many
// of photons as there are to each (two, on a Yee grid and a standing wave one), in turn, which
// keeps loads in flight beside both halves of the leptons.  Against a launch each, same device:
// 64-electron cascade 3124 to 2860 us, mixed cascade 28.0 to 26.2 ms, 64 mixed instances 14.4
// to 12.7, grid cascade 35.3 to 32.3, largest rotating cascade 141 to 128 (leptons first
// throughout: 136; in turn throughout: 64 instances 13.3, grid 33.3).
// kInterleave and the exception: where a photon's field is evaluated and not loaded (a standing
// wave), arithmetic bounds the photons too, and leptons first is faster at every ratio (FP64,
// first / in turn: 8 times the photons 350 / 359 us a step, 16 times 337 / 400, 80 times 413 /
// 436).  Elsewhere the measured ratios disagree by form (8 times: grid 424 / 500, rotating 246 /
// 252, uniform B 280 / 289, its mixed form 278 / 272; 16 times: grid 1311 / 1258, rotating 236 /
// 239, uniform B 275 / 270; 80 times: mixed rotating 345 / 342, mixed uniform 358 / 333), and the
// largest rotating cascade, 128 ms with 8, takes 137 with 16 and 136 with 32.
constexpr long long kInterleave = 8;
template <bool MIXED, int FMODE>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(LeptonShape<MIXED, FMODE, false>::min_waves)))
    particle_kernel(StepArgs a, int lep_grid, int pho_grid) {
  __shared__ union Lds {
    LeptonLds<MIXED, FMODE, false> lep;
    PhotonLds pho;
    __device__ Lds() {}
  } lds;
  // cycles of one group of lepton workgroups and `per` of photon ones; then the other leptons,
  // then the other photons, and last the lepton workgroups without work
  const int b = (int)blockIdx.x, group = a.cus;
  const int lep_work = lepton_blocks(a);
  const int per = max(pho_grid / lep_work, 1);
  const bool loads = FMODE != kFieldLocal || a.field.kind == QED_FIELD_YEE;
  const int cycles = loads && a.hdr->pho_total >= kInterleave * a.hdr->lep_total
                         ? min(lep_work / group, pho_grid / (group * per))
                         : 0;
  Place at;
  bool lep;
  const int r = b - cycles * (1 + per) * group;
  if (r < 0) {
    const int g = b / group, c = g / (1 + per), w = g - c * (1 + per);
    lep = w == 0;
    at.block = (lep ? c : c * per + w - 1) * group + (b - g * group);
  } else {
    const int more = lep_work - cycles * group, pho = pho_grid - cycles * per * group;
    lep = r < more || r >= more + pho;
    at.block = r < more ? cycles * group + r
               : lep    ? lep_work + (r - more - pho)
                        : cycles * per * group + (r - more);
  }
  at.grid = lep ? lep_work : pho_grid;
  if (lep) lepton_step<MIXED, FMODE, false, false>(a, at, lds.lep);
  // (one batch where a second bought nothing: a position-dependent field, whose loads come back
  // after the batches ahead of them, and the mixed rotating form: its cascade 26.03 ms, 26.24
  // with two, though 80 photons a lepton take 323 us with two and 335 with one)
  else photon_step<MIXED, FMODE,
                   FMODE == kFieldLocal || (MIXED && FMODE == kFieldE) ? 1 : 2>(a, at, lds.pho);
}

// State of one wavefront of the exact pair-decision kernel.
struct ExactCtx {
  Series64 ser64;
  Series32 ser32;
  FieldArgs fld;
  uint32_t step;
  int wid;
  int staged;
  ArenaCursor acur;  // this wavefront's place in the pair arena
  ArenaTally tally;
  const double* bound;  // per-octave pair-rate bounds (LDS)
  const MathTab* mt;    // (LDS)
};

// The pair records of the lanes with `make` into the wavefront's arena share or pool chunks,
// else staged and reserved in the stores (an electron and a positron each); all lanes call.
// `sub` is the sub-step code (sub-step and run), `later` whether the pair has time left in
// the step.
template <int FMODE>
__device__ __forceinline__ void exact_append(const StepArgs& a, ExactCtx& c, PairStage& ps,
                                             LaneCounters& cnt, WaveCounters& wc, bool make,
                                             const V3& x, const V3& kv, double r1, double wp,
                                             uint64_t id, uint32_t sub, int inst, double tau,
                                             const V3& Ef, const V3& Bf, bool later) {
  const uint64_t below = lanes_below();
  const uint64_t pm = wave_ballot(make);
  if (!pm) return;
  const int n_new = __popcll(pm);
  wc.events += n_new;
  const ChildArena& qa = a.qa;
  ArenaSpan span;
  if (qa.waves > 0 && arena_reserve(qa, c.wid, c.acur, n_new, span)) {
    // ---- pair records into the wavefront's arena share or pool chunks ----
    c.tally.add(qa, c.wid, pm, make, inst);
    if (make) {
      const long long r = span.at(__popcll(pm & below));
      qa.x[r] = x.x;
      qa.y[r] = x.y;
      qa.z[r] = x.z;
      qa.px[r] = kv.x;
      qa.py[r] = kv.y;
      qa.pz[r] = kv.z;
      qa.r1[r] = r1;
      qa.w[r] = wp;
      qa.parent[r] = id;
      qa.sub[r] = sub;
      qa.inst[r] = (unsigned)inst;
      if (a.generations > 0) record_same_step<FMODE>(qa, r, tau, Ef, Bf);
    }
    return;
  }
  // reserved directly in the stores: not advanced in this step (an electron and a positron)
  if (a.generations > 0) wc.deferred += 2 * __popcll(wave_ballot(later));
  // ---- else stage them and reserve e-/e+ slots once per batch ----
  if (c.staged + n_new > kStageCap) {
    flush_pairs(a, ps, c.staged, c.step, cnt);
    c.staged = 0;
  }
  if (make) {
    const int r = c.staged + __popcll(pm & below);
    ps.x[r] = x.x;
    ps.y[r] = x.y;
    ps.z[r] = x.z;
    ps.kx[r] = kv.x;
    ps.ky[r] = kv.y;
    ps.kz[r] = kv.z;
    ps.r1[r] = r1;
    ps.w[r] = wp;
    ps.parent[r] = id;
    ps.sub[r] = sub;
    ps.inst[r] = inst;
  }
  c.staged += n_new;
}

// One candidate of the photon kernel's lists, re-derived from the stores: its slot, instance,
// columns, fields and setup, and the sub-step kc its draw fell below the bound at.
struct ExactCand {
  long long s;
  int inst, kc;
  uint64_t id, seed;
  V3 x, kv, E, B;
  PhotonSetup st;
};

template <bool MIXED, int FMODE>
__device__ __forceinline__ ExactCand load_candidate(const StepArgs& a, const ExactCtx& c,
                                                    unsigned long long e) {
  const qed_soa& S = a.sp[QED_PHOTON];
  ExactCand q;
  const long long g = (long long)(e >> 16);
  q.kc = (int)(e & 0xFFFFull);
  int lo = 0, hi = a.n_inst;  // pho_pref[lo] <= g < pho_pref[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (a.pho_pref[mid] <= g) lo = mid;
    else hi = mid;
  }
  q.inst = lo;
  q.s = a.inst[q.inst].base[QED_PHOTON] + (g - a.pho_pref[q.inst]);
  q.id = S.id[q.s];
  q.x = {S.x[q.s], S.y[q.s], S.z[q.s]};
  q.kv = {S.px[q.s], S.py[q.s], S.pz[q.s]};
  const Root kr = root_of(dot(q.kv, q.kv));
  const double kabs = kr.r, inv_k = kr.under(1.0);
  q.seed = a.inst[q.inst].seed;
  if (FMODE == kFieldLocal) field_at_position<true>(c.fld, a.inst[q.inst].amp, q.x, q.E, q.B);
  else instance_fields<FMODE>(a, q.inst, q.E, q.B);
  q.st = photon_setup<MIXED, FMODE != kFieldE>(a, q.E, q.B, q.kv, kabs, inv_k, c.bound, nullptr);
  return q;
}

// Exact pair decision for the candidate `entry` of each lane that has one; all lanes call.
template <bool MIXED, int FMODE>
__device__ __forceinline__ void exact_batch(const StepArgs& a, ExactCtx& c, PairStage& ps,
                                            LaneCounters& cnt, WaveCounters& wc, bool has,
                                            unsigned long long entry) {
  const qed_soa& S = a.sp[QED_PHOTON];
  bool pair = false, make = false;
  double r1 = 0.0, wp = 0.0, tau = 0.0;
  int kpair = 0, inst = 0, nsub = 0;
  V3 x{}, kv{}, Ef{}, Bf{};
  uint64_t id = 0;
  if (has) {
    const ExactCand q = load_candidate<MIXED, FMODE>(a, c, entry);
    const PhotonSetup& st = q.st;
    const long long s = q.s;
    inst = q.inst;
    id = q.id;
    x = q.x;
    kv = q.kv;
    int done = st.nsub;
    for (int k = 0; k < st.nsub; ++k) {
      if (a.push_photons) x = {x.x + st.hk * kv.x, x.y + st.hk * kv.y, x.z + st.hk * kv.z};
      if (k < q.kc) continue;  // settled by the bound in photon_kernel
      const uint4 o = draw_words(id, q.seed, c.step, (uint32_t)k, kDraw);
      if (k > q.kc && !below_bound<MIXED>(o, st.pbound)) {
        ++cnt.early;
        continue;
      }
      if (pair_decision<MIXED>(a, *c.mt, c.ser64, c.ser32, o, st.chi, st.pref, cnt, &r1)) {
        pair = true;
        kpair = k;
        done = k + 1;
        break;
      }
    }
    cnt.subs += done - q.kc;
    if (a.push_photons) {
      S.x[s] = x.x;
      S.y[s] = x.y;
      S.z[s] = x.z;
    }
    if (pair) {
      // the photon decays at every event; with a generator factor f_g (Sec. VI) the pair is
      // created with probability 1 / f_g, or for one photon in f_g in the deterministic
      // form, and carries f_g times the photon's weight
      S.id[s] = QED_ID_DEAD;
      make = a.every_pair     ? generator_every(id, q.seed, 0u, a.every_pair)
             : a.fg_pair > 1.0 ? generator_runs(id, q.seed, c.step, (uint32_t)kpair, kGenPair,
                                                a.inv_fg_pair)
                               : true;
      wp = S.w[s] * a.fg_pair;
      nsub = st.nsub;
      tau = (double)(st.nsub - kpair - 1) * st.h;
      Ef = q.E;
      Bf = q.B;
    }
  }
  exact_append<FMODE>(a, c, ps, cnt, wc, make, x, kv, r1, wp, id, (uint32_t)kpair, inst, tau,
                      Ef, Bf, make && kpair < nsub - 1);
}

// The same in the reverse mode of Sec. VI (N_g = runs_pair > 1): the photon stands for N_g
// copies of weight w / N_g.  Lanes go through their sub-steps together from the candidate's
// kc; at each, every run draws (the bound settles most), each run that fires makes a pair of
// the copies' weight, the photon keeps the weight of the copies left and is removed when all
// N_g fire.  Pairs are appended run by run, so a photon can make several.
template <bool MIXED, int FMODE>
__device__ __forceinline__ void exact_batch_runs(const StepArgs& a, ExactCtx& c, PairStage& ps,
                                                 LaneCounters& cnt, WaveCounters& wc, bool has,
                                                 unsigned long long entry) {
  const qed_soa& S = a.sp[QED_PHOTON];
  const int R = a.runs_pair;
  bool live = has;
  ExactCand q{};
  int k = 0;
  double wcur = 0.0;
  if (live) {
    q = load_candidate<MIXED, FMODE>(a, c, entry);
    // the sub-steps before kc were settled by the bound: only the push remains
    if (a.push_photons)
      for (; k < q.kc; ++k)
        q.x = {q.x.x + q.st.hk * q.kv.x, q.x.y + q.st.hk * q.kv.y, q.x.z + q.st.hk * q.kv.z};
    k = q.kc;
    wcur = S.w[q.s];
  }
  while (wave_ballot(live)) {
    double wc_run = 0.0;
    if (live) {
      if (a.push_photons)
        q.x = {q.x.x + q.st.hk * q.kv.x, q.x.y + q.st.hk * q.kv.y, q.x.z + q.st.hk * q.kv.z};
      wc_run = wcur / (double)R;
    }
    int m = 0;
    const double tau = live ? (double)(q.st.nsub - k - 1) * q.st.h : 0.0;
    for (int run = 0; run < R; ++run) {
      bool make = false;
      double r1 = 0.0;
      const uint32_t sc = sub_code(k, run);
      if (live) {
        const uint4 o = draw_words(q.id, q.seed, c.step, sc, kDraw);
        if (!below_bound<MIXED>(o, q.st.pbound)) ++cnt.early;
        else make = pair_decision<MIXED>(a, *c.mt, c.ser64, c.ser32, o, q.st.chi, q.st.pref, cnt, &r1);
        m += make;
      }
      exact_append<FMODE>(a, c, ps, cnt, wc, make, q.x, q.kv, r1, wc_run, q.id, sc, q.inst, tau,
                          q.E, q.B, make && k < q.st.nsub - 1);
    }
    if (live) {
      ++k;
      ++cnt.subs;
      const bool dead = m == R;
      if (!dead && m > 0) wcur = wc_run * (double)(R - m);
      if (dead || k == q.st.nsub) {
        live = false;
        if (a.push_photons) {
          S.x[q.s] = q.x.x;
          S.y[q.s] = q.x.y;
          S.z[q.s] = q.x.z;
        }
        if (dead) S.id[q.s] = QED_ID_DEAD;
        else if (wcur != S.w[q.s]) S.w[q.s] = wcur;
      }
    }
  }
}

// Candidate lists of one workgroup at most (the lists of kMaxWaves photon wavefronts over
// kExactGridBlocks workgroups); one wavefront scans their counts.
constexpr int kExactLists = (kMaxWaves + kExactGridBlocks - 1) / kExactGridBlocks;
static_assert(kExactLists < 64, "one wavefront scans a workgroup's list counts");

template <bool MIXED, int FMODE, bool RUNS>
__device__ __forceinline__ void exact_pass(const StepArgs& a) {
  __shared__ BlockStats bs;
  __shared__ PairStage pstage[kWavesPerBlock];
  __shared__ double sbound[kBoundEntries];
  __shared__ MathTab mt;
  __shared__ unsigned lfirst[kExactLists + 1];  // first candidate of each list of the workgroup
  WorkHdr* hdr = a.hdr;
  const int wpb = (int)(blockDim.x >> 6);
  // The photon kernel's per-wavefront lists are cut over the workgroups, and a workgroup's
  // candidates are one index space, 64 at a time per wavefront: the lists hold a few each, and
  // a wavefront that took list after list waited for the columns of each in turn (mixed
  // cascade, 14.2 to 11.4 us a launch; 9.4 to 3 where there is no candidate).
  const long long chunk = chunk_size(hdr->pho_total, a.pho_waves, a.pho_deal);
  const int lists = (int)working_waves(hdr->pho_total, a.pho_waves, chunk);
  const int per = (lists + (int)gridDim.x - 1) / (int)gridDim.x;  // <= kExactLists
  const int l0 = (int)blockIdx.x * per < lists ? (int)blockIdx.x * per : lists;
  const int nl = l0 + per < lists ? per : lists - l0;
  if (threadIdx.x < 64) {
    const int l = (int)threadIdx.x;
    const unsigned v = l < nl ? a.candn[l0 + l] : 0u;
    unsigned x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned y = __shfl_up(x, o, 64);
      if (l >= o) x += y;
    }
    if (l <= kExactLists) lfirst[l] = x - v;
  }
  __syncthreads();
  const int n_lists = (int)lfirst[nl];
  long long n_over = (long long)hdr->n_cand;  // the overflow list
  if (n_over > a.cand_cap) n_over = a.cand_cap;
  if (n_lists == 0 && n_over == 0) {
    if (a.qa.waves > 0 && lane_id() == 0) a.qa.nrec[wave_index()] = 0u;
    for (int i = threadIdx.x; i < kPfNsub; i += blockDim.x)
      a.ex_part[part_index(i, (int)blockIdx.x)] = 0ull;
    return;
  }
  block_stats_init(bs);
  stage_bounds<MIXED>(a, sbound);
  if (!MIXED) stage_math(mt);  // (the FP32 rates use the hardware's log2 and exp)
  __syncthreads();
  ExactCtx c;
  c.bound = sbound;
  c.mt = &mt;
  c.ser64 = {a.tables->series[0], a.tables->series[1], a.tables->series[2], a.tables->series[3],
             a.tables->series[4]};
  c.ser32 = {(float)c.ser64.b0, (float)c.ser64.b1, (float)c.ser64.c0, (float)c.ser64.c1,
             (float)c.ser64.c2};
  c.fld = a.field;
  c.fld.tn = hdr->tn;
  c.step = (uint32_t)hdr->step;
  c.wid = wave_index();
  c.staged = 0;
  c.acur = ArenaCursor{};
  PairStage& ps = pstage[threadIdx.x >> 6];
  LaneCounters cnt;
  cnt.bs = &bs;
  WaveCounters wc;
  const int V = (int)gridDim.x * (int)(blockDim.x >> 6);

  for (int i0 = (int)(threadIdx.x & ~63u); i0 < n_lists; i0 += wpb * 64) {
    const int i = i0 + lane_id();
    unsigned long long e = 0ull;
    if (i < n_lists) {
      int lo = 0, hi = nl;  // lfirst[lo] <= i < lfirst[hi]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((int)lfirst[mid] <= i) lo = mid;
        else hi = mid;
      }
      e = a.candw[(size_t)(l0 + lo) * a.cand_per_wave + (size_t)(i - (int)lfirst[lo])];
    }
    if constexpr (RUNS) exact_batch_runs<MIXED, FMODE>(a, c, ps, cnt, wc, i < n_lists, e);
    else exact_batch<MIXED, FMODE>(a, c, ps, cnt, wc, i < n_lists, e);
  }
  // then the overflow list
  for (long long i0 = (long long)c.wid * 64; i0 < n_over; i0 += (long long)V * 64) {
    const bool has = i0 + lane_id() < n_over;
    const unsigned long long e = has ? a.cand[i0 + lane_id()] : 0ull;
    if constexpr (RUNS) exact_batch_runs<MIXED, FMODE>(a, c, ps, cnt, wc, has, e);
    else exact_batch<MIXED, FMODE>(a, c, ps, cnt, wc, has, e);
  }

  if (c.staged > 0) flush_pairs(a, ps, c.staged, c.step, cnt);
  if (a.qa.waves > 0) {
    c.tally.flush(a.qa, c.wid);
    if (lane_id() == 0) a.qa.nrec[c.wid] = (unsigned)c.acur.n;
  }
  wave_to_block(bs, cnt, wc);
  __syncthreads();
  block_stats_store(bs, a.ex_part, kPfNsub, (int)blockIdx.x);
}

template <bool MIXED, int FMODE>
__global__ void __launch_bounds__(256) photon_exact_kernel(StepArgs a) {
  exact_pass<MIXED, FMODE, false>(a);
}

// The reverse mode of Sec. VI (runs_pair > 1) in a kernel of its own, for the registers,
// held to two wavefronts per SIMD.
template <bool MIXED, int FMODE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
    photon_exact_runs_kernel(StepArgs a) {
  exact_pass<MIXED, FMODE, true>(a);
}

// ------------------------------------------------------------------------------------
// arena append: scan of the per-(instance, wavefront) counts, then the copy into the stores
// ------------------------------------------------------------------------------------
// Exclusive prefix over n words by a workgroup of 1024: thread t sums the run [t k, t k + k),
// one scan of the thread sums, then the run's offsets in place.  Returns the total; `wsum` is
// 16 words of LDS.
__device__ __forceinline__ unsigned long long block_prefix(unsigned int* row, int n,
                                                           unsigned long long* wsum) {
  const int lane = lane_id();
  const int wv = (int)(threadIdx.x >> 6);
  const int nw = (int)(blockDim.x >> 6);
  const int k = (n + (int)blockDim.x - 1) / (int)blockDim.x;
  const int j0 = (int)threadIdx.x * k;
  const int j1 = j0 + k < n ? j0 + k : n;
  unsigned long long v = 0ull;
  for (int j = j0; j < j1; ++j) v += row[j];
  unsigned long long x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wv] = x;
  __syncthreads();
  unsigned long long run = x - v, carry = 0;
  for (int q = 0; q < nw; ++q) {
    if (q < wv) run += wsum[q];
    carry += wsum[q];
  }
  for (int j = j0; j < j1; ++j) {
    const unsigned c = row[j];
    row[j] = (unsigned)run;
    run += c;
  }
  __syncthreads();  // wsum is taken again
  return carry;
}

// Two workgroups per instance, photons and pairs (4.7 us a launch; 6.7 with one taking both in
// turn): exclusive prefix over the wavefronts of the arena's counts (in place), the store
// count before the append into base[], and the counts raised by the totals, clamped to the
// capacities; the copy kernel drops and counts the children that land beyond them.
// With same-step processing (A.slot set) one more workgroup turns each arena's record counts
// per producing wavefront into their prefix, and the total goes to used[1], so that the next
// generation's wavefronts find the records they are dealt.  `in_p`, `in_q`: totals of the
// records that the producing generation read (null: not one): where both are 0 it made none,
// and only the totals are set.
__global__ void __launch_bounds__(1024) arena_scan_kernel(StepArgs a, ChildArena pa,
                                                          ChildArena qa,
                                                          const unsigned int* in_p,
                                                          const unsigned int* in_q) {
  __shared__ unsigned long long wsum[16];
  const int i = (int)blockIdx.x >> 1;
  const bool none = in_p && *in_p == 0u && *in_q == 0u;
  if (i == a.n_inst) {
    for (int kind = 0; kind < 2; ++kind) {
      const ChildArena& A = kind == 0 ? pa : qa;
      if (A.waves <= 0) continue;
      const unsigned long long total = none ? 0ull : block_prefix(A.nrec, A.waves, wsum);
      if (threadIdx.x == 0) A.used[1] = (unsigned)total;
    }
    return;
  }
  if (none) return;
  const int kind = (int)(blockIdx.x & 1u);  // photons, pairs
  const ChildArena& A = kind == 0 ? pa : qa;
  unsigned long long total = 0ull;
  if (A.waves > 0) total = block_prefix(A.cnt + (size_t)i * A.waves, A.waves, wsum);
  if (threadIdx.x != 0) return;
  // the store counts before the append, and the new ones; counts above the capacity (the copy
  // drops and counts what lands beyond it) are clamped
  qed_instance& I = a.inst[i];
  const int s0 = kind == 0 ? QED_PHOTON : QED_ELECTRON, s1 = kind == 0 ? QED_PHOTON : QED_POSITRON;
  for (int s = s0; s <= s1; ++s) {
    const long long before = I.count[s];
    if (A.waves > 0) A.base[2 * i + (s - s0)] = before;
    const long long after = before + (long long)total;
    I.count[s] = after > I.capacity[s] ? I.capacity[s] : after;
  }
}

// Count n children dropped for lack of capacity (rare: only at a full store).
__device__ __forceinline__ void count_drops(const StepArgs& a, int inst, bool lost) {
  uint64_t m = wave_ballot(lost);
  while (m) {
    const int leader = __ffsll((unsigned long long)m) - 1;
    const int li = wave_bcast(inst, leader);
    const uint64_t same = wave_ballot(lost && inst == li);
    if (lane_id() == leader) {
      atomicAdd(reinterpret_cast<unsigned long long*>(&a.inst[li].dropped),
                (unsigned long long)__popcll(same));
      atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats->dropped),
                (unsigned long long)__popcll(same));
      atomicOr(&a.stats->status, QED_STATUS_DROPPED);
    }
    m &= ~same;
  }
}

// Records of producing wavefront sw (after the scan).
__device__ __forceinline__ long long wave_records(const ChildArena& A, int sw) {
  if (!A.slot) return (long long)A.nrec[sw];
  const unsigned end = sw + 1 < A.waves ? A.nrec[sw + 1] : A.used[1];
  return (long long)(end - A.nrec[sw]);
}

// One wavefront per producing wavefront: walks its records in order and gives each the
// next store slot of its instance after the offsets of the scan (a per-instance running
// count in LDS), then writes the child (photon) or both children (pair record), and, for
// same-step processing, the slots into the record.  The launch also clears the count
// matrices of the arenas zpa, zqa (the next generation's, whose readers are done).  When
// the step has no later producer, its first reduce_blocks workgroups take the partial-stats
// reduction instead (the reduce kernel's jobs), and the launch ends the step: the scan has
// clamped the counts and the status bits are set where their counters are raised, so only
// the step counter is left to advance (no kernel of this launch reads it).
__global__ void __launch_bounds__(256) arena_copy_kernel(StepArgs a, ChildArena pa,
                                                         ChildArena qa, ChildArena zpa,
                                                         ChildArena zqa, int reduce_blocks) {
  __shared__ unsigned int lcnt[kWavesPerBlock][kArenaMaxInstances];
  if ((int)blockIdx.x < reduce_blocks) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.d_step = a.hdr->step + 1;
    reduce_job(a, (int)blockIdx.x * kWavesPerBlock + (int)(threadIdx.x >> 6), lane_id());
    return;
  }
  const int blk = (int)blockIdx.x - reduce_blocks;  // the copy's own workgroups
  const int nblk = (int)gridDim.x - reduce_blocks;
  {
    const long long n1 = zpa.waves > 0 ? (long long)a.n_inst * zpa.waves : 0;
    const long long n2 = zqa.waves > 0 ? (long long)a.n_inst * zqa.waves : 0;
    const long long stride = (long long)nblk * blockDim.x;
    for (long long i = (long long)blk * blockDim.x + threadIdx.x; i < n1 + n2; i += stride) {
      if (i < n1) zpa.cnt[i] = 0u;
      else zqa.cnt[i - n1] = 0u;
    }
    if (blk == 0 && threadIdx.x == 0) {
      if (zpa.waves > 0) *zpa.used = 0u;
      if (zqa.waves > 0) *zqa.used = 0u;
    }
  }
  unsigned int* run = lcnt[threadIdx.x >> 6];
  const uint64_t below = lanes_below();
  const int lane = lane_id();
  const uint32_t step = (uint32_t)a.hdr->step;
  const int npa = pa.waves > 0 && !(pa.slot && pa.used[1] == 0u) ? pa.waves : 0;
  const int nqa = qa.waves > 0 && !(qa.slot && qa.used[1] == 0u) ? qa.waves : 0;
  const int V = nblk * (int)(blockDim.x >> 6);
  const int wid = blk * (int)(blockDim.x >> 6) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  for (int t = wid; t < npa + nqa; t += V) {
    const bool pair = t >= npa;
    const ChildArena& A = pair ? qa : pa;
    const int sw = pair ? t - npa : t;
    const long long n = wave_records(A, sw);
    if (n == 0) continue;
    if (a.n_inst > 1)
      for (int q = lane; q < a.n_inst; q += 64) run[q] = 0u;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    ArenaWalk walk;
    for (long long j0 = 0; j0 < n; j0 += 64) {
      const long long j = j0 + lane;
      const bool has = j < n;
      walk.advance(A, sw, j0, 64, n);
      const long long r = has ? walk.index(A, sw, j) : 0;
      const int li = has ? (int)A.inst[r] : -1;
      unsigned local = (unsigned)j;  // one instance: the record's place in the wavefront's
      uint64_t m = a.n_inst > 1 ? wave_ballot(has) : 0ull;
      while (m) {
        const int leader = __ffsll((unsigned long long)m) - 1;
        const int lj = wave_bcast(li, leader);
        const uint64_t same = wave_ballot(has && li == lj);
        const unsigned c0 = run[lj];
        if (has && li == lj) local = c0 + (unsigned)__popcll(same & below);
        __builtin_amdgcn_wave_barrier();
        if (lane == leader) run[lj] = c0 + (unsigned)__popcll(same);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        m &= ~same;
      }
      bool lost0 = false, lost1 = false;
      if (has) {
        const qed_instance& I = a.inst[li];
        const long long off = (long long)A.cnt[(size_t)li * A.waves + sw] + local;
        const uint64_t seed = I.seed;
        // each record is read once (non-temporal loads: 20.2 to 18.4 us a launch)
        const uint32_t sub = __builtin_nontemporal_load(&A.sub[r]);
        const uint64_t parent = __builtin_nontemporal_load(&A.parent[r]);
        const double x = __builtin_nontemporal_load(&A.x[r]);
        const double y = __builtin_nontemporal_load(&A.y[r]);
        const double z = __builtin_nontemporal_load(&A.z[r]);
        const double px = __builtin_nontemporal_load(&A.px[r]);
        const double py = __builtin_nontemporal_load(&A.py[r]);
        const double pz = __builtin_nontemporal_load(&A.pz[r]);
        const double w = __builtin_nontemporal_load(&A.w[r]);
        if (!pair) {
          const long long d = A.base[2 * li] + off;
          if (d < I.capacity[QED_PHOTON]) {
            const qed_soa& o = a.sp[QED_PHOTON];
            const long long q = I.base[QED_PHOTON] + d;
            o.x[q] = x;
            o.y[q] = y;
            o.z[q] = z;
            o.px[q] = px;
            o.py[q] = py;
            o.pz[q] = pz;
            o.w[q] = w;
            o.id[q] = child_id(parent, seed, step, sub, kPhotonChild);
            o.parent[q] = parent;
            o.birth[q] = birth_code(step, sub);
            if (o.n_events) o.n_events[q] = 0u;
            if (A.slot) A.slot[r] = q;
          } else {
            lost0 = true;
            if (A.slot) A.slot[r] = -1;
          }
        } else {
          // electron takes r1 of the photon momentum, positron the rest (Sec. V.A)
          const double r1 = A.r1[r];
          const double r1c = 1.0 - r1;
          const long long de = A.base[2 * li] + off;
          if (de < I.capacity[QED_ELECTRON]) {
            const qed_soa& o = a.sp[QED_ELECTRON];
            const long long q = I.base[QED_ELECTRON] + de;
            o.x[q] = x;
            o.y[q] = y;
            o.z[q] = z;
            o.px[q] = r1 * px;
            o.py[q] = r1 * py;
            o.pz[q] = r1 * pz;
            o.w[q] = w;
            o.id[q] = child_id(parent, seed, step, sub, kElectronChild);
            o.parent[q] = parent;
            o.birth[q] = birth_code(step, sub);
            if (o.n_events) o.n_events[q] = 0u;
            if (A.slot) A.slot[r] = q;
          } else {
            lost0 = true;
            if (A.slot) A.slot[r] = -1;
          }
          const long long dp = A.base[2 * li + 1] + off;
          if (dp < I.capacity[QED_POSITRON]) {
            const qed_soa& o = a.sp[QED_POSITRON];
            const long long q = I.base[QED_POSITRON] + dp;
            o.x[q] = x;
            o.y[q] = y;
            o.z[q] = z;
            o.px[q] = r1c * px;
            o.py[q] = r1c * py;
            o.pz[q] = r1c * pz;
            o.w[q] = w;
            o.id[q] = child_id(parent, seed, step, sub, kPositronChild);
            o.parent[q] = parent;
            o.birth[q] = birth_code(step, sub);
            if (o.n_events) o.n_events[q] = 0u;
            if (A.slot2) A.slot2[r] = q;
          } else {
            lost1 = true;
            if (A.slot2) A.slot2[r] = -1;
          }
        }
      }
      if (wave_ballot(lost0 || lost1)) {
        count_drops(a, li, lost0);
        count_drops(a, li, lost1);
      }
    }
  }
}

// ------------------------------------------------------------------------------------
// children in their birth step (same-step processing)
// ------------------------------------------------------------------------------------
// A generation pass reads the records the previous pass (or the step's particle kernels)
// wrote and the copy kernel placed in the stores, advances each child in its store slot
// through the time it has left in the step, with its parent's frozen fields, and writes the
// children it creates to the other arena set (with their own time left), from where the
// next scan and copy place them.  Generations alternate between the two sets.
struct GenArgs {
  ChildArena ipa, iqa;  // input: photon records and pair records of the previous pass
  ChildArena opa, oqa;  // output: this kernel's wavefronts write their children here
  int pass;             // 1 .. G
  int last;             // 1 on pass G: what it creates waits for the next step
};
// kernel arguments stay within the 4 KB the launch passes
static_assert(sizeof(StepArgs) + sizeof(GenArgs) <= 4096, "generation kernel arguments");
static_assert(sizeof(StepArgs) + 4 * sizeof(ChildArena) + 8 <= 4096, "copy kernel arguments");

// Fields a child inherited from its parent (record r of A).
template <int FMODE>
__device__ __forceinline__ void inherited_fields(const StepArgs& a, const ChildArena& A,
                                                 long long r, int inst, V3& E, V3& B) {
  if (FMODE == kFieldLocal) {
    const long long c = A.cap;
    const double* f = A.fe;
    E = {f[r], f[c + r], f[2 * c + r]};
    B = {f[3 * c + r], f[4 * c + r], f[5 * c + r]};
  } else {
    instance_fields<FMODE>(a, inst, E, B);
  }
}

struct GenWave {
  int wid;
  ArenaCursor cp, cq;  // this wavefront's place in opa, oqa
  ArenaTally tp, tq;
};

// A wavefront's stream of children: all records of arena A in the order of their producing
// wavefronts are one index space, one item per photon record or two (electron, positron) per
// pair record, dealt in chunks over the V wavefronts.  The children of one parent, or of one
// busy wavefront, thus spread over the whole GPU: a generation lasts as long as the longest
// chain of sub-steps, where wavefronts that took over the records of one producer each ran
// through hundreds of chains while the others were idle (the large-step shower of 125 seeds,
// three steps: 47.9 to 19.5 ms).
struct GenStream {
  long long n = 0, j = 0, jend = 0, next_chunk = 0, V = 1;
  int c = 1;  // items of a chunk
  bool pair = false;
  __device__ __forceinline__ void init(const ChildArena& A, int wid, int v, bool is_pair) {
    V = v;
    pair = is_pair;
    n = A.waves > 0 ? (pair ? 2 : 1) * (long long)A.used[1] : 0;
    const long long per = n / (4 * V);
    c = per < 1 ? 1 : per > 64 ? 64 : (int)per;
    next_chunk = wid;
  }
  // The next piece [j0, j0 + take), take <= want <= 64; false once the stream is exhausted.
  // Wavefront-uniform; all lanes call.
  __device__ __forceinline__ bool next(int want, long long& j0, int& take) {
    if (j >= jend) {
      j = next_chunk * c;
      if (j >= n) return false;
      jend = j + c < n ? j + c : n;
      next_chunk += V;
    }
    take = (int)((long long)want < jend - j ? (long long)want : jend - j);
    j0 = j;
    j += take;
    return true;
  }
  // Record holding item jj.
  __device__ __forceinline__ long long record(const ChildArena& A, long long jj) const {
    const unsigned i = (unsigned)(pair ? jj >> 1 : jj);
    int lo = 0, hi = A.waves;  // nrec[lo] <= i < nrec[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (A.nrec[mid] <= i) lo = mid;
      else hi = mid;
    }
    long long k = (long long)(i - A.nrec[lo]);
    if (k < A.per_wave) return (long long)lo * A.per_wave + k;
    k -= A.per_wave;
    unsigned chunk = A.first[lo];
    for (; k >= kArenaChunk; k -= kArenaChunk) chunk = A.next[chunk];
    return A.pool0 + (long long)chunk * kArenaChunk + k;
  }
};

// Electrons and positrons of the input pair records, each advanced through its tau; a lane
// whose lepton has done all its sub-steps takes the next one from the wavefront's stream.
template <bool MIXED, int FMODE, bool RUNS>
__device__ __forceinline__ void gen_lepton_phase(const StepArgs& a, const GenArgs& q,
                                                 GenWave& gw, int V,
                                                 const typename TabType<MIXED>::T* tab,
                                                 const MathTab& mt, const Series64& ser64,
                                                 const Series32& ser32, BlockStats& bs,
                                                 LaneCounters& cnt, WaveCounters& wc) {
  const ChildArena& A = q.iqa;
  const ChildArena& O = q.opa;
  const uint64_t below = lanes_below();
  const uint32_t step = (uint32_t)a.hdr->step;
  GenStream st;
  st.init(A, gw.wid, V, true);
  long long slot = -1;
  int sp = 0, inst = 0;
  LepLane L;
  V3 &x = L.x, &p = L.p, &E = L.E, &B = L.B;
  int &k = L.k, &left = L.left;
  double &h = L.h;
  uint64_t id = 0, seed = 0;
  double wgt = 0.0;
  uint32_t nev = 0;
  const bool refine = a.forced <= 0 && a.adaptive;
  while (true) {
    // ---- refill idle lanes ----
    uint64_t freem = wave_ballot(slot < 0);
    while (freem) {
      long long j0;
      int take;
      if (!st.next(__popcll(freem), j0, take)) break;
      const int rank = __popcll(freem & below);
      bool act = false;
      if (slot < 0 && rank < take) {
        const long long jj = j0 + rank;
        const long long r = st.record(A, jj);
        const long long sl = (jj & 1) ? A.slot2[r] : A.slot[r];
        const double tau = A.tau[r];
        if (sl >= 0 && tau > 0.0) {
          act = true;
          sp = (jj & 1) ? QED_POSITRON : QED_ELECTRON;
          inst = (int)A.inst[r];
          x = {LEPTON_COL(x, sp)[sl], LEPTON_COL(y, sp)[sl], LEPTON_COL(z, sp)[sl]};
          p = {LEPTON_COL(px, sp)[sl], LEPTON_COL(py, sp)[sl], LEPTON_COL(pz, sp)[sl]};
          id = LEPTON_COL(id, sp)[sl];
          wgt = LEPTON_COL(w, sp)[sl];
          uint32_t* ne = LEPTON_COL(n_events, sp);
          nev = ne ? ne[sl] : 0u;
          seed = a.inst[inst].seed;
          inherited_fields<FMODE>(a, A, r, inst, E, B);
          const Kin kn = kin_of<FMODE != kFieldE>(p, E, B);
          int nsub = 1;
          if (a.forced > 0) {
            nsub = a.forced;
          } else if (a.adaptive && kn.c2 > 0.0) {
            const NsubInfo ni =
                nsub_from_ratio(substep_ratio_lepton(mt, tau, kn, a.eps_r, a.inv_lep_scale));
            nsub = ni.n;
            if (ni.near_int) block_count(bs, kPfNearInt);
            if (ni.clamped) block_count(bs, kPfClamped);
          }
          if (!isfinite(kn.c2)) block_count(bs, kPfNonfinite);
          h = div_normal(tau, (double)nsub, rcp_normal((double)nsub));
          L.dtfac = h * a.dtfac_per_h;
          L.qh2 = (sp == QED_ELECTRON ? -0.5 : 0.5) * h;
          L.hs3 = a.eps_r * a.eps_r * substep_cube(h, a.inv_lep_scale);
          k = 0;
          left = nsub;
          slot = sl;
        }
      }
      wc.children += __popcll(wave_ballot(act));
      freem = wave_ballot(slot < 0);
    }
    if (wave_ballot(slot >= 0) == 0) break;

    // ---- one sub-step, with the first run of the emission generator ----
    Kin kn{0.0, 0.0, {1.0, 1.0, true}};
    bool first = false;
    double delta1 = 0.0;
    for (;;) {  // (until a lane emits or ends its last sub-step, as in lepton_step)
      if (slot >= 0) {
        first = lepton_substep<MIXED, FMODE != kFieldE>(a, tab, mt, ser64, ser32, id, seed,
                                                        step, refine, L, kn, bs, cnt, delta1);
        ++cnt.subs;
      }
      if (RUNS || wave_ballot(slot >= 0 && (first || left == 1))) break;
      ++k;
      --left;
    }
    // the emission generator, N_g times in the reverse mode of Sec. VI (as in lepton_step)
    const int runs = RUNS ? a.runs_photon : 1;
    const double wrun = wgt / (double)runs;
    V3 rec = {0.0, 0.0, 0.0};
    bool fired = false;
    for (int run = 0; run < runs; ++run) {
      const uint32_t sc = sub_code(k, run);
      bool emit = false;
      double f = 0.0;
      if (slot >= 0 && a.emission) {
        double delta = delta1;
        if (run == 0)
          emit = first;
        else
          emit = emission_decision<MIXED>(
              tab, mt, ser64, ser32, emission_draw<MIXED>(draw_words(id, seed, step, sc, kDraw)),
              kn, a.eps_r, a.z_scale, L.dtfac, cnt, delta);
        if (emit) {
          emit = emission_photon(mt, kn, delta, wrun, bs, cnt, f);
          if (emit) ++nev;
        }
      }
      bool child = emit;
      if (emit) {
        if (a.every_photon) child = generator_every(id, seed, nev - 1u, a.every_photon);
        else if (a.fg_photon > 1.0)
          child = generator_runs(id, seed, step, (uint32_t)k, kGenPhoton, a.inv_fg_photon);
      }
      const uint64_t em = wave_ballot(child);
      if (em) {
        const int n_new = __popcll(em);
        wc.events += n_new;
        const double cw = runs > 1 ? wrun : wgt * a.fg_photon;
        const bool later = child && left > 1;  // the photon has time left in the step
        ArenaSpan span;
        if (O.waves > 0 && arena_reserve(O, gw.wid, gw.cp, n_new, span)) {
          gw.tp.add(O, gw.wid, em, child, inst);
          if (child) {
            const long long rr = span.at(__popcll(em & below));
            O.x[rr] = x.x;
            O.y[rr] = x.y;
            O.z[rr] = x.z;
            O.px[rr] = f * p.x;
            O.py[rr] = f * p.y;
            O.pz[rr] = f * p.z;
            O.w[rr] = cw;
            O.parent[rr] = id;
            O.sub[rr] = sc;
            O.inst[rr] = (unsigned)inst;
            record_same_step<FMODE>(O, rr, (double)(left - 1) * h, E, B);
          }
          if (q.last) wc.deferred += __popcll(wave_ballot(later));
        } else {
          // the arena is full: reserved directly, not advanced in this step
          wave_append<QED_PHOTON>(a, child, inst, cnt, [&](const qed_soa& o, long long s2) {
            o.x[s2] = x.x;
            o.y[s2] = x.y;
            o.z[s2] = x.z;
            o.px[s2] = f * p.x;
            o.py[s2] = f * p.y;
            o.pz[s2] = f * p.z;
            o.w[s2] = cw;
            o.id[s2] = child_id(id, seed, step, sc, kPhotonChild);
            o.parent[s2] = id;
            o.birth[s2] = birth_code(step, (uint32_t)k);
            if (o.n_events) o.n_events[s2] = 0u;
          });
          wc.deferred += __popcll(wave_ballot(later));
        }
      }
      if (emit) {
        // recoil: the lepton keeps p - k (momentum conservation, Sec. IV.F)
        if (runs == 1) {
          p = recoil(p, f);
        } else {
          rec = {rec.x + f * p.x, rec.y + f * p.y, rec.z + f * p.z};
          fired = true;
        }
      }
    }
    if (fired) {
      const double R = (double)runs;
      p = {p.x - rec.x / R, p.y - rec.y / R, p.z - rec.z / R};
    }
    if (slot >= 0 && (++k, --left == 0)) {
      LEPTON_COL(x, sp)[slot] = x.x;
      LEPTON_COL(y, sp)[slot] = x.y;
      LEPTON_COL(z, sp)[slot] = x.z;
      LEPTON_COL(px, sp)[slot] = p.x;
      LEPTON_COL(py, sp)[slot] = p.y;
      LEPTON_COL(pz, sp)[slot] = p.z;
      uint32_t* ne = LEPTON_COL(n_events, sp);
      if (ne) ne[slot] = nev;
      slot = -1;
    }
  }
}

// Photons of the input photon records, each advanced through its tau (lane refill as for
// the leptons).
template <bool MIXED, int FMODE, bool RUNS>
__device__ __forceinline__ void gen_photon_phase(const StepArgs& a, const GenArgs& q,
                                                 GenWave& gw, int V, const MathTab& mt,
                                                 const Series64& ser64, const Series32& ser32,
                                                 BlockStats& bs, LaneCounters& cnt,
                                                 LaneCounters& pcnt, WaveCounters& wc) {
  const ChildArena& A = q.ipa;
  const ChildArena& O = q.oqa;
  const uint64_t below = lanes_below();
  const uint32_t step = (uint32_t)a.hdr->step;
  const qed_soa& S = a.sp[QED_PHOTON];
  const bool photons = a.push_photons || a.pairs;
  GenStream st;
  // from the last wavefront on, so that few photons and few leptons meet on none
  st.init(A, V - 1 - gw.wid, V, false);
  long long slot = -1;
  int inst = 0, nsub = 0, k = 0;
  uint64_t id = 0, seed = 0;
  V3 x{}, kv{}, E{}, B{};
  double chi = 0.0, h = 0.0, hk = 0.0, pref = 0.0, wcur = 0.0;
  while (true) {
    // ---- refill idle lanes ----
    uint64_t freem = wave_ballot(slot < 0);
    while (freem) {
      long long j0;
      int take;
      if (!st.next(__popcll(freem), j0, take)) break;
      const int rank = __popcll(freem & below);
      bool act = false;
      if (slot < 0 && rank < take) {
        const long long r = st.record(A, j0 + rank);
        const long long sl = A.slot[r];
        const double tau = A.tau[r];
        act = sl >= 0 && tau > 0.0;
        if (act && photons) {
          id = S.id[sl];
          x = {S.x[sl], S.y[sl], S.z[sl]};
          kv = {S.px[sl], S.py[sl], S.pz[sl]};
          const Root kr = root_of(dot(kv, kv));
          const double kabs = kr.r, inv_k = kr.under(1.0);
          if (!(kabs > 0.0) || !isfinite(kabs)) {
            block_count(bs, kPfNonfinite);
          } else {
            inst = (int)A.inst[r];
            seed = a.inst[inst].seed;
            inherited_fields<FMODE>(a, A, r, inst, E, B);
            chi = a.eps_r * root_of(chi_sq<FMODE != kFieldE>(kv, kabs, E, B)).r;
            nsub = 1;
            if (a.forced > 0) {
              nsub = a.forced;
            } else if (a.adaptive && chi > 0.0) {
              // tau / dt_q with dt_q of Eq. (33)
              const NsubInfo ni = nsub_from_ratio(tau * (chi * inv_k) * a.inv_pho_scale);
              nsub = ni.n;
              if (ni.near_int) block_count(bs, kPfNearInt);
              if (ni.clamped) block_count(bs, kPfClamped);
            }
            if (!isfinite(chi)) block_count(bs, kPfNonfinite);
            h = nsub == 1 ? tau : div_normal(tau, (double)nsub, rcp_normal((double)nsub));
            hk = h * inv_k;
            pref = h * (a.dtfac_per_h * kInvSqrt3Pi) * inv_k;
            wcur = S.w[sl];
            k = 0;
            slot = sl;
          }
        }
      }
      wc.children += __popcll(wave_ballot(act));
      freem = wave_ballot(slot < 0);
    }
    if (wave_ballot(slot >= 0) == 0) break;

    // ---- one sub-step: the pair generator once, or N_g times in the reverse mode of
    // Sec. VI (as in the exact pass) ----
    const int R = RUNS ? a.runs_pair : 1;
    int m = 0;
    if (slot >= 0) {
      if (a.push_photons) x = {x.x + hk * kv.x, x.y + hk * kv.y, x.z + hk * kv.z};
      ++cnt.subs;
    }
    const double wc_run = R > 1 ? wcur / (double)R : wcur;
    for (int run = 0; run < R; ++run) {
      const uint32_t sc = sub_code(k, run);
      bool make = false;
      double r1 = 0.0, wp = 0.0;
      if (slot >= 0 && a.pairs) {
        const uint4 o = draw_words(id, seed, step, sc, kDraw);
        if (pair_decision<MIXED>(a, mt, ser64, ser32, o, chi, pref, pcnt, &r1)) {
          ++m;
          // the photon decays; its pair is created with probability 1 / f_g, or for one
          // photon in f_g in the deterministic form (Sec. VI)
          make = R > 1           ? true
                 : a.every_pair  ? generator_every(id, seed, 0u, a.every_pair)
                 : a.fg_pair > 1.0 ? generator_runs(id, seed, step, (uint32_t)k, kGenPair,
                                                    a.inv_fg_pair)
                                   : true;
          wp = R > 1 ? wc_run : wcur * a.fg_pair;
        }
      }
      const uint64_t pm = wave_ballot(make);
      if (!pm) continue;
      const int n_new = __popcll(pm);
      wc.pairs += n_new;
      const bool later = make && k < nsub - 1;
      ArenaSpan span;
      if (O.waves > 0 && arena_reserve(O, gw.wid, gw.cq, n_new, span)) {
        gw.tq.add(O, gw.wid, pm, make, inst);
        if (make) {
          const long long rr = span.at(__popcll(pm & below));
          O.x[rr] = x.x;
          O.y[rr] = x.y;
          O.z[rr] = x.z;
          O.px[rr] = kv.x;
          O.py[rr] = kv.y;
          O.pz[rr] = kv.z;
          O.r1[rr] = r1;
          O.w[rr] = wp;
          O.parent[rr] = id;
          O.sub[rr] = sc;
          O.inst[rr] = (unsigned)inst;
          record_same_step<FMODE>(O, rr, (double)(nsub - k - 1) * h, E, B);
        }
        if (q.last) wc.deferred += 2 * __popcll(wave_ballot(later));
      } else {
        // the arena is full: reserved directly, not advanced in this step
        const double r1c = 1.0 - r1;
        wave_append<QED_ELECTRON>(a, make, inst, cnt, [&](const qed_soa& o, long long s2) {
          o.x[s2] = x.x;
          o.y[s2] = x.y;
          o.z[s2] = x.z;
          o.px[s2] = r1 * kv.x;
          o.py[s2] = r1 * kv.y;
          o.pz[s2] = r1 * kv.z;
          o.w[s2] = wp;
          o.id[s2] = child_id(id, seed, step, sc, kElectronChild);
          o.parent[s2] = id;
          o.birth[s2] = birth_code(step, (uint32_t)k);
          if (o.n_events) o.n_events[s2] = 0u;
        });
        wave_append<QED_POSITRON>(a, make, inst, cnt, [&](const qed_soa& o, long long s2) {
          o.x[s2] = x.x;
          o.y[s2] = x.y;
          o.z[s2] = x.z;
          o.px[s2] = r1c * kv.x;
          o.py[s2] = r1c * kv.y;
          o.pz[s2] = r1c * kv.z;
          o.w[s2] = wp;
          o.id[s2] = child_id(id, seed, step, sc, kPositronChild);
          o.parent[s2] = id;
          o.birth[s2] = birth_code(step, (uint32_t)k);
          if (o.n_events) o.n_events[s2] = 0u;
        });
        wc.deferred += 2 * __popcll(wave_ballot(later));
      }
    }
    if (slot >= 0) {
      const bool dead = m == R;  // every copy decayed
      if (!dead && m > 0) wcur = wc_run * (double)(R - m);
      if (dead || ++k == nsub) {
        if (a.push_photons) {
          S.x[slot] = x.x;
          S.y[slot] = x.y;
          S.z[slot] = x.z;
        }
        if (dead) S.id[slot] = QED_ID_DEAD;
        else if (wcur != S.w[slot]) S.w[slot] = wcur;
        slot = -1;
      }
    }
  }
}

// Is any wavefront of this workgroup dealt one of n items (of the lepton or the photon stream)?
__device__ __forceinline__ bool gen_block_has_work(long long n, bool leptons) {
  const long long wpb = blockDim.x >> 6, V = (long long)gridDim.x * wpb;
  const long long per = n / (4 * V);
  const long long c = per < 1 ? 1 : per > 64 ? 64 : per;
  const long long first = leptons ? (long long)blockIdx.x * wpb
                                  : V - ((long long)blockIdx.x + 1) * wpb;
  return first * c < n;
}

template <bool MIXED, int FMODE, bool RUNS>
__device__ __forceinline__ void gen_pass(const StepArgs& a, const GenArgs& q) {
  using Tab = typename TabType<MIXED>::T;
  __shared__ BlockStats bs;
  __shared__ Tab tab[kTableN];  // the emission table, as in the lepton kernel
  __shared__ MathTab mt;
  // a workgroup without a child writes its empty counts (only the first pass stores its
  // statistics; the scan takes a generation without children at all as empty)
  const unsigned np = q.ipa.waves > 0 ? q.ipa.used[1] : 0u;
  const unsigned nq = q.iqa.waves > 0 ? q.iqa.used[1] : 0u;
  if (np == 0u && nq == 0u) {
    if (q.pass > 1) return;
  }
  const bool work = gen_block_has_work(np, false) || gen_block_has_work(2ll * nq, true);
  if (!work) {
    if (lane_id() == 0) {
      if (q.opa.waves > 0) q.opa.nrec[wave_index()] = 0u;
      if (q.oqa.waves > 0) q.oqa.nrec[wave_index()] = 0u;
    }
    if (q.pass == 1)
      for (int i = threadIdx.x; i < kPfCount; i += blockDim.x)
        a.gen_part[part_index(i, (int)blockIdx.x)] = 0ull;
    return;
  }
  block_stats_init(bs);
  stage_math(mt);
  {
    const Tab* src = MIXED ? reinterpret_cast<const Tab*>(a.tables->ab32)
                           : reinterpret_cast<const Tab*>(a.tables->ab64);
    for (int i = threadIdx.x; i < kTableN; i += blockDim.x) tab[i] = src[i];
  }
  __syncthreads();
  const Series64 ser64 = {a.tables->series[0], a.tables->series[1], a.tables->series[2],
                          a.tables->series[3], a.tables->series[4]};
  const Series32 ser32 = {(float)ser64.b0, (float)ser64.b1, (float)ser64.c0, (float)ser64.c1,
                          (float)ser64.c2};
  const int lane = lane_id();
  const int V = (int)gridDim.x * (int)(blockDim.x >> 6);
  GenWave gw;
  gw.wid = wave_index();
  LaneCounters cnt, pcnt;  // pcnt: pair decisions
  cnt.bs = &bs;
  pcnt.bs = &bs;
  WaveCounters wc;
  // photons of the previous generation, then its electrons and positrons
  gen_photon_phase<MIXED, FMODE, RUNS>(a, q, gw, V, mt, ser64, ser32, bs, cnt, pcnt, wc);
  gen_lepton_phase<MIXED, FMODE, RUNS>(a, q, gw, V, tab, mt, ser64, ser32, bs, cnt, wc);
  if (q.opa.waves > 0) {
    gw.tp.flush(q.opa, gw.wid);
    if (lane == 0) q.opa.nrec[gw.wid] = (unsigned)gw.cp.n;
  }
  if (q.oqa.waves > 0) {
    gw.tq.flush(q.oqa, gw.wid);
    if (lane == 0) q.oqa.nrec[gw.wid] = (unsigned)gw.cq.n;
  }
  wave_to_block(bs, cnt, wc, &pcnt);
  __syncthreads();
  block_stats_accumulate(bs, a.gen_part, q.pass == 1);
}

template <bool MIXED, int FMODE>
__global__ void __launch_bounds__(256) gen_kernel(StepArgs a, GenArgs q) {
  gen_pass<MIXED, FMODE, false>(a, q);
}

// The reverse mode of Sec. VI (runs_photon or runs_pair > 1) in a kernel of its own.
template <bool MIXED, int FMODE>
__global__ void __launch_bounds__(256) gen_runs_kernel(StepArgs a, GenArgs q) {
  gen_pass<MIXED, FMODE, true>(a, q);
}

#undef LEPTON_COL

// ------------------------------------------------------------------------------------
// Returns whether the arena copy took the partial-stats reduction and ended the step (no
// producer after it).
template <bool MIXED, int FMODE>
static bool launch_persistent(const StepArgs& a, LaunchShape lep, LaunchShape pho,
                              bool run_photons, hipStream_t s) {
  const bool ext = a.generations > 0 || a.fg_photon > 1.0;
  if (a.events[0]) (void)hipEventRecord(a.events[0], s);
  if (a.one_launch)
    hipLaunchKernelGGL((particle_kernel<MIXED, FMODE>), dim3(lep.grid + pho.grid),
                       dim3(lep.block), 0, s, a, lep.grid, pho.grid);
  else if (a.runs_photon > 1)
    hipLaunchKernelGGL((lepton_runs_kernel<MIXED, FMODE>), dim3(lep.grid), dim3(lep.block), 0,
                       s, a);
  else if (ext)
    hipLaunchKernelGGL((lepton_kernel<MIXED, FMODE, true>), dim3(lep.grid), dim3(lep.block), 0,
                       s, a);
  else
    hipLaunchKernelGGL((lepton_kernel<MIXED, FMODE, false>), dim3(lep.grid), dim3(lep.block), 0,
                       s, a);
  if (a.events[1]) (void)hipEventRecord(a.events[1], s);
  if (run_photons && !a.one_launch) {
    if (a.events[2]) (void)hipEventRecord(a.events[2], s);
    hipLaunchKernelGGL((photon_kernel<MIXED, FMODE>), dim3(pho.grid), dim3(pho.block), 0, s, a);
    if (a.events[3]) (void)hipEventRecord(a.events[3], s);
  }
  if (run_photons) {
    if (a.ex_grid > 0 && a.runs_pair > 1)
      hipLaunchKernelGGL((photon_exact_runs_kernel<MIXED, FMODE>), dim3(a.ex_grid), dim3(256), 0,
                         s, a);
    else if (a.ex_grid > 0)
      hipLaunchKernelGGL((photon_exact_kernel<MIXED, FMODE>), dim3(a.ex_grid), dim3(256), 0, s, a);
  }
  const int src = a.pa.waves + a.qa.waves;
  const ChildArena none{};
  const bool gen = a.generations > 0;
  const int rb = gen ? 0 : reduce_blocks(a);
  if (src > 0) {
    const unsigned int* no = nullptr;
    hipLaunchKernelGGL(arena_scan_kernel, dim3(2 * a.n_inst + (gen ? 1 : 0)), dim3(1024), 0, s, a,
                       a.pa, a.qa, no, no);
    // with same-step processing the copy also clears generation 1's count matrices
    hipLaunchKernelGGL(arena_copy_kernel,
                       dim3(rb + (src + kWavesPerBlock - 1) / kWavesPerBlock), dim3(256), 0, s,
                       a, a.pa, a.qa, gen ? a.gpa[1] : none, gen ? a.gqa[1] : none, rb);
  }
  // children through the rest of the step: generation g reads set (g - 1) % 2 (set 0 as the
  // particle kernels wrote it for g = 1) and writes set g % 2
  for (int g = 1; g <= a.generations; ++g) {
    GenArgs q;
    q.ipa = g == 1 ? a.pa : a.gpa[(g - 1) % 2];
    q.iqa = g == 1 ? a.qa : a.gqa[(g - 1) % 2];
    q.opa = a.gpa[g % 2];
    q.oqa = a.gqa[g % 2];
    q.pass = g;
    q.last = g == a.generations ? 1 : 0;
    if (a.runs_photon > 1 || a.runs_pair > 1)
      hipLaunchKernelGGL((gen_runs_kernel<MIXED, FMODE>), dim3(a.gen_grid), dim3(256), 0, s, a, q);
    else
      hipLaunchKernelGGL((gen_kernel<MIXED, FMODE>), dim3(a.gen_grid), dim3(256), 0, s, a, q);
    const int gsrc = q.opa.waves + q.oqa.waves;
    const bool more = g < a.generations;
    // (both input arenas are on, or the photon one alone: its total then serves twice)
    const unsigned int* in_p = q.ipa.used + 1;
    const unsigned int* in_q = q.iqa.waves > 0 ? q.iqa.used + 1 : in_p;
    hipLaunchKernelGGL(arena_scan_kernel, dim3(2 * a.n_inst + 1), dim3(1024), 0, s, a, q.opa, q.oqa,
                       in_p, in_q);
    hipLaunchKernelGGL(arena_copy_kernel, dim3((gsrc + kWavesPerBlock - 1) / kWavesPerBlock),
                       dim3(256), 0, s, a, q.opa, q.oqa, more ? a.gpa[(g + 1) % 2] : none,
                       more ? a.gqa[(g + 1) % 2] : none, 0);
  }
  return src > 0 && !gen;
}

int field_mode(int kind) {
  if (kind == QED_FIELD_UNIFORM) return kFieldEB;
  if (kind == QED_FIELD_ROTATING_E) return kFieldE;
  return kFieldLocal;
}

hipError_t launch_step(const StepArgs& a, int precision, LaunchShape lep, LaunchShape pho,
                       bool run_photons, hipStream_t s) {
  const long long zero_words = (long long)a.n_inst * (a.pa.waves + a.qa.waves);
  long long zb = (zero_words + 2047) / 2048;
  if (zb > 1024) zb = 1024;
  hipLaunchKernelGGL(prep_kernel, dim3(1 + (int)zb), dim3(256), 0, s, a, run_photons ? 1 : 0);
  const int fm = field_mode(a.field.kind);
  bool reduced;
  if (precision == QED_MIXED) {
    if (fm == kFieldEB) reduced = launch_persistent<true, kFieldEB>(a, lep, pho, run_photons, s);
    else if (fm == kFieldE) reduced = launch_persistent<true, kFieldE>(a, lep, pho, run_photons, s);
    else reduced = launch_persistent<true, kFieldLocal>(a, lep, pho, run_photons, s);
  } else {
    if (fm == kFieldEB) reduced = launch_persistent<false, kFieldEB>(a, lep, pho, run_photons, s);
    else if (fm == kFieldE) reduced = launch_persistent<false, kFieldE>(a, lep, pho, run_photons, s);
    else reduced = launch_persistent<false, kFieldLocal>(a, lep, pho, run_photons, s);
  }
  if (!reduced) {
    hipLaunchKernelGGL(reduce_kernel, dim3(reduce_blocks(a)), dim3(256), 0, s, a);
    hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

// Resident workgroups per CU of a step kernel: kind 0 the photon kernel, 1 the lepton
// kernel, 2 its extended form, 3 its reverse-mode form, 4 the kernel of both.
template <bool MIXED, int FMODE>
static int occupancy(int kind, int block) {
  int nb = 0;
  hipError_t e;
  if (kind == 0)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, photon_kernel<MIXED, FMODE>, block, 0);
  else if (kind == 4)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, particle_kernel<MIXED, FMODE>, block, 0);
  else if (kind == 3)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, lepton_runs_kernel<MIXED, FMODE>,
                                                     block, 0);
  else if (kind == 2)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, lepton_kernel<MIXED, FMODE, true>,
                                                     block, 0);
  else
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, lepton_kernel<MIXED, FMODE, false>,
                                                     block, 0);
  return (e != hipSuccess || nb < 1) ? 1 : nb;
}

template <bool MIXED>
static int occupancy_of(int fmode, int kind, int block) {
  if (fmode == kFieldEB) return occupancy<MIXED, kFieldEB>(kind, block);
  if (fmode == kFieldE) return occupancy<MIXED, kFieldE>(kind, block);
  return occupancy<MIXED, kFieldLocal>(kind, block);
}

int step_blocks_per_cu(int precision, int fmode, int kind, int block) {
  return precision == QED_MIXED ? occupancy_of<true>(fmode, kind, block)
                                : occupancy_of<false>(fmode, kind, block);
}

}  // namespace qedk
