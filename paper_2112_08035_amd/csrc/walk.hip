// walk.hip -- the persistent photon-packet walk through an SDF scene on
// gfx950 (McMillan, Bruce & Dholakia 2021, Sec. 2.3), one packet per lane.
//
// Each lane owns a packet: emission (Sec. 3.1 sources, Eq. 1 free path),
// sphere-tracing steps over every region SDF (Sec. 2.3, Fig. 3), the
// interface step in FP64 (Fresnel, numerical normals; Sec. 1 and Sec. 2.3),
// interactions (implicit capture, Henyey-Greenstein, roulette), and the
// path-length fluence tally (Sec. 3.1, rectangular bins).  When its packet
// ends the lane takes the next packet id from a global counter, so the grid
// is sized to the machine, not to the packet count.
//
// T is the transport type (float or double): positions, directions, step
// lengths, the SDFs of the stepping loop and the transcendentals.  The
// interface step, remaining optical depth, weights, absorbed energy and
// tallies are FP64 in both.  Steps may be over-relaxed (a multiple of the
// surface distance, checked at the next evaluation; Sec. 5).
//
// Divergence control: packets that reach a surface wait until surface_min / 64
// of the wave's packets are there, and the wave then takes up to eight of them
// through the long FP64 interface step together, eight lanes each; dead lanes
// wait for refill_min (or for a wave without packets) before a wave emits.
//
// Tally: a lane keeps the straight path since its last tally pending and
// credits it through the voxel grid (a register-only DDA) before an
// interaction, an interface event or the packet's end.  Consecutive pieces
// in the same voxel (across steps, events and even packets) merge into one
// run; each run is staged in the wave's LDS stage, which is drained as
// full-wave FP64 atomics.
#include <hip/hip_runtime.h>

#include <climits>

#include "launch.h"
#include "voxel_model.h"
#include "walk_common.h"

namespace smcrt {

// ---- interface steps.  A packet within delta of a surface needs, in FP64:
// the nearest region, its numerical normal, the hit where the ray meets it,
// the normal there, and a probe across it for the medium ahead; then it
// crosses, reflects or refracts.  The region SDFs of these points are nearly
// all of the work, and only a few lanes of a wave are at a surface at a time.
// So the wave shares it: eight lanes per packet, eight packets per step.  The
// lanes of a group evaluate the regions side by side, then the six points of
// each central difference side by side -- four evaluations in a row instead
// of 2 n_regions + 12 -- through one copy of the SDF code (40 KB of kernel
// instead of 200 KB, which the instruction cache does not hold).  Every SDF
// is the one the packet's own lane would compute.  Against each lane doing its
// own: 5e5 packets of a 2000-capsule network 25 % less time, 1e6 of the 256^3
// cylinder 7 %, 1e7 of the slab the same (its interface steps are a small
// share and its tally atomics bound it).

// value of lane k of the caller's group of eight
__device__ __forceinline__ double group_get(double x, int group, int k) {
  return __shfl(x, (group << 3) + k);
}

// fence between the lanes of one wave (LDS records)
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// region_dist<double> of a region that differs between lanes.  Scenes with
// placed primitives take the regions one after the other, so that their many
// parameters stay scalar loads.
template <bool XF>
__device__ __forceinline__ double lane_region_dist(JobRef a, int r, V3<double> p) {
  if constexpr (XF) {
    double d = 0.0;
    for (bool todo = true; todo;) {
      const int r0 = __builtin_amdgcn_readfirstlane(r);
      if (r == r0) {
        d = region_dist<double, XF>(a, r0, p);
        todo = false;
      }
    }
    return d;
  } else {
    return region_dist<double, XF>(a, r, p);
  }
}

// The geometry of the interface steps in slots [0, n): in, the packets'
// positions, directions and regions; out, the ray's way to the surface, the
// surface point, the normal there, its cosine with the direction, and the
// region across.  Called with every lane of the wave active.  What a step
// hands to the next stays in the slot: held in registers, it pushed the walk
// over its register budget.
template <bool XF>
__device__ __forceinline__ void surface_geometry(JobRef a, SurfaceSlot* S, int n, int lane) {
  ScP sc = fresh(kptr(a.sc));
  const int group = lane >> 3, sub = lane & 7;
  const bool on = group < n, first = on && sub == 0;
  SurfaceSlot& s = S[on ? group : 0];
  const int nr = sc->n_regions;
  double dj = 0.0;
  int j = 0, r2 = nr;
  // steps: the regions' distances at p (eight regions at a time), the
  // normal at p, the normal at the surface point, the regions at the probe
  const int rounds = (nr + 7) >> 3;
  for (int step = 0; step < 2 * rounds + 2; ++step) {
    const bool nearest = step < rounds, probe = step >= rounds + 2;
    const int base = nearest ? 8 * step : (probe ? 8 * (step - rounds - 2) : 0);
    int r = base + sub;
    V3<double> q = mk(s.p[0], s.p[1], s.p[2]);
    bool eval = on && r < nr;
    if (probe) {
      const double sg = s.c > 0.0 ? 1.0 : -1.0;
      q = q + (sg * sc->offset) * mk(s.u[0], s.u[1], s.u[2]);
    } else if (!nearest) {
      // the points of the central differences: +x -x +y -y +z -z
      const double h = sc->h_normal;
      const double e = (sub & 1) ? -h : h;
      r = j;
      q.x = sub < 2 ? q.x + e : q.x;
      q.y = (sub & 6) == 2 ? q.y + e : q.y;
      q.z = (sub & 6) == 4 ? q.z + e : q.z;
      eval = on && sub < 6;
    }
    double d = 0.0;
    if (eval) d = lane_region_dist<XF>(a, r, q);
    if (nearest) {
      const int m = nr - base < 8 ? nr - base : 8;
      for (int k = 0; k < m; ++k) {
        const double dk = group_get(d, group, k);
        if (base + k == 0 || __builtin_fabs(dk) < __builtin_fabs(dj)) {
          dj = dk;
          j = base + k;
        }
      }
    } else if (probe) {
      const uint64_t neg = __ballot(eval && d < 0.0);
      const uint32_t mine = (uint32_t)(neg >> (group << 3)) & 0xffu;
      if (mine) r2 = base + 31 - __clz(mine);
    } else {
      V3<double> g;
      g.x = group_get(d, group, 0) - group_get(d, group, 1);
      g.y = group_get(d, group, 2) - group_get(d, group, 3);
      g.z = group_get(d, group, 4) - group_get(d, group, 5);
      const double inv = 1.0 / __builtin_sqrt(dot(g, g));
      g = inv * g;
      const V3<double> u = mk(s.u[0], s.u[1], s.u[2]);
      const double c = dot(u, g);
      V3<double> ps = mk(s.p[0], s.p[1], s.p[2]);
      double t_ray = 0.0;
      if (step == rounds) {  // at p: where the ray meets the surface
        if (__builtin_fabs(c) >= sc->snap_cos) {
          t_ray = -dj / c;
          ps = ps + t_ray * u;
        } else {
          ps = ps - dj * g;
        }
      }
      wave_fence();
      if (first) {
        if (step == rounds) {
          s.p[0] = ps.x; s.p[1] = ps.y; s.p[2] = ps.z;
          s.t_ray = t_ray;
        } else {
          s.u[0] = g.x; s.u[1] = g.y; s.u[2] = g.z;
          s.c = c;
        }
      }
      wave_fence();
    }
  }
  if (first && s.c != 0.0) s.region = r2;
  wave_fence();
}

// The packet's way to its surface.  Returns true when it stands on an
// interface (its event follows in surface_event, once its path is tallied);
// else pk.state is set: it moved on (no change of medium ahead) or interacts
// before the surface.
template <typename T>
__device__ __forceinline__ bool surface_arrive(JobRef a, Regions<T> rg, const SurfaceSlot& s, Packet<T>& pk, LdsTallies& L) {
  ScP sc = fresh(kptr(a.sc));
  const double mut = rg[pk.region].mut;
  const double off = sc->offset, t_ray = s.t_ray;
  double tau = pk.tau;
  const double s_rem = mut > 0.0 ? tau / mut : __builtin_inf();
  if (s.region == pk.region) {
    // no change of medium ahead: advance 2*delta along the ray
    atomicAdd(&L.cnt[kCAdvances], 1ull);
    if (s_rem <= off) {
      advance(pk, (T)s_rem);
      pk.tau = 0.0;
      pk.state = kInteract;
      return false;
    }
    advance(pk, (T)off);
    pk.tau = tau - mut * off;
    pk.state = kTransport;
    return false;
  }
  if (t_ray > 0.0) {
    if (s_rem <= t_ray) {
      advance(pk, (T)s_rem);
      pk.tau = 0.0;
      pk.state = kInteract;
      return false;
    }
    advance(pk, (T)t_ray);
    tau -= mut * t_ray;
  }
  pk.tau = tau;
  pk.state = kTransport;
  return true;
}

// The change of medium at the surface: cross, reflect or refract.
template <typename T, bool TRACE>
__device__ __forceinline__ void surface_event(JobRef a, Regions<T> rg, const SurfaceSlot& s, Packet<T>& pk, Lane& ln, LdsTallies& L) {
  ScP sc = fresh(kptr(a.sc));
  const V3<double> u = to_d(pk.u), ps = mk(s.p[0], s.p[1], s.p[2]), nrm = mk(s.u[0], s.u[1], s.u[2]);
  const double off = sc->offset, c = s.c;
  const double sg = c > 0.0 ? 1.0 : -1.0;
  const V3<double> q = ps + (sg * off) * nrm;
  const int r2 = s.region;
  pk.k += 1;
  pk.steps = 0;
  pk.pd = T(-1);
  atomicAdd(&L.cnt[kCInterfaces], 1ull);
  const double n1 = rg[pk.region].n, n2 = rg[r2].n;
  if (n1 == n2) {  // index matched: cross undeflected
    set_position(pk, q);
    set_region(rg, pk, r2);
    atomicAdd(&L.cnt[kCCrossings], 1ull);
    record<T, TRACE>(a, pk, ln, SMCRT_EV_CROSS);
    return;
  }
  const U4 rr = philox10(pk.k, (uint32_t)pk.pid, (uint32_t)(pk.pid >> 32), 0u, (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
  const double x0 = xi_of<double>(rr.w0);
  const double ci = __builtin_fabs(c), eta = n1 / n2;
  double ctr;
  const double R = fresnel(n1, n2, ci, &ctr);
  V3<double> v;
  if (x0 < R) {  // specular reflection, back on the incident side
    v = u - (2.0 * c) * nrm;
    set_position(pk, ps - (sg * off) * nrm);
    v = (1.0 / __builtin_sqrt(dot(v, v))) * v;
    pk.u = from_d<T>(v);
    atomicAdd(&L.cnt[kCReflections], 1ull);
    record<T, TRACE>(a, pk, ln, SMCRT_EV_REFLECT);
  } else {  // refraction (vector Snell's law) into the far medium
    v = eta * u + ((ctr - eta * ci) * sg) * nrm;
    v = (1.0 / __builtin_sqrt(dot(v, v))) * v;
    pk.u = from_d<T>(v);
    set_position(pk, q);
    set_region(rg, pk, r2);
    atomicAdd(&L.cnt[kCRefractions], 1ull);
    record<T, TRACE>(a, pk, ln, SMCRT_EV_REFRACT);
  }
}

constexpr int kDueMin = 32;  // see the sphere-tracing steps

// The persistent walk over a table of jobs (scene tables, seed, packet
// range, outputs).  Each wave works on one job at a time, so the job's
// tables are wave uniform and come through the scalar cache; waves start
// spread over the jobs in proportion to their count and, when their job's
// packets are all handed out and their lanes have drained, flush their sums
// into that job's outputs and move on to the next job with packets left.
// GEOM selects the geometry model: sphere tracing through the SDFs, or the
// voxel walk of the voxelised comparison model.  XF adds the path of placed,
// modified and further-shape primitives.  The launch takes only the jobs of
// its (GEOM, XF) class.  4 waves per SIMD in FP32 (3 in FP64) keep the
// walk's state in registers.
//
// STAGE (FP32, scenes whose accelerated region is plain capsules): the
// workgroup is 16 waves, one per SIMD slot of a CU, that work on one job
// together.  It copies the job's capsule records into an LDS table once per
// job, so the grid queries of the step loop -- a gather of a few capsules
// per lane per step -- read LDS instead of global memory; the waves meet at
// a barrier when the job is drained, and the workgroup takes the next job
// and its table together.
//
// EPOCH (resident serving): the launch stops at B.deadline, saving the
// packets in flight, and resumes the jobs' saved packets before taking new
// ids.  A separate instantiation: the save and resume paths cost registers
// the plain walk does not spend.
//
// SEG (kLaunchSegment jobs): over-relaxed steps (in the XF kernels too) or, for
// segment-tracing scenes: every evaluation also bounds the way along the
// ray to each region's surface (segment tracing), and a step runs to the
// nearest such bound less delta when that is longer than the distance.
template <typename T, bool TRACE, int GEOM, bool XF, bool STAGE, bool EPOCH, bool SEG>
__global__ void __launch_bounds__(STAGE ? 1024 : 256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 3)))
walk_kernel(const WalkArgs* __restrict__ job_table, BatchArgs B) {
  static_assert(!STAGE || (sizeof(T) == 4 && GEOM == kGeomSdf && !XF && !TRACE), "staged capsules: FP32 SDF walks");
  static_assert(!EPOCH || !TRACE, "epochs are for runs, not traces");
  static_assert(!SEG || (GEOM == kGeomSdf && !XF && !STAGE), "segment tracing: plain SDF walks");
  constexpr int kWaves = STAGE ? 16 : 4;
  constexpr bool kRelax = SEG || XF;  // kernels whose scenes may take over-relaxed steps
  const SMCRT_K WalkArgs* jobs = kptr(job_table);
  __shared__ LdsTallies Lw[kWaves];
  __shared__ WaveStage Sw[kWaves];
  __shared__ SurfaceSlot Hw[GEOM == kGeomSdf ? kWaves : 1][kSurfaceSlots];
  LdsCaps caps_lds = nullptr;
  F4* caps_fill = nullptr;
  int* wg_job = nullptr;
  uint64_t* wg_t0 = nullptr;
  if constexpr (STAGE) {
    __shared__ F4 s_caps[2 * kStageCaps];
    __shared__ int s_job;
    __shared__ uint64_t s_t0;
    caps_lds = (LdsCaps)s_caps;
    caps_fill = s_caps;
    wg_job = &s_job;
    wg_t0 = &s_t0;
  }
  // the region table of the wave's job (of the workgroup's, when staged)
  __shared__ RegionRow<T> Rw[STAGE ? 1 : kWaves][kMaxRegions + 1];
  const int lane = lane_id();
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave index in the block (wave uniform)
  LdsTallies& L = Lw[wib];
  RegionRow<T>* rows = Rw[STAGE ? 0 : wib];
  const Regions<T> rg = (Regions<T>)rows;
  clear_tallies(L, lane);

  Lane ln;
  ln.stage = &Sw[wib];
  ln.run.v = -1;
  ln.run.sum = 0.0;
  ln.abs_sum = 0.0;
  ln.abs_region = -1;
  ln.n_steps = ln.n_inter = 0;
  ln.rec = nullptr;
  ln.n_rec = 0;
  WaveTally wt = {0, 0ull, 0ull};

  // resident serving: a launch with a deadline stops when the device wall
  // clock has run deadline ticks past its start (the workgroup's start in
  // the staged kernel, so that its waves agree), saving the packets still
  // in flight for the next epoch
  uint64_t t0 = 0;
  bool stop = false;
  if constexpr (EPOCH && !STAGE) t0 = __builtin_amdgcn_s_memrealtime();

  // First jobs, XCD-aware: workgroups go to the 8 XCDs in turn (block b to
  // XCD b mod 8), and each XCD has its own L2.  The jobs are split into 8
  // runs of consecutive jobs, one per XCD, and every workgroup of an XCD
  // starts at the first job of its run; a job that runs out sends its
  // workgroups on to the next one (pick_job scans forward).  So an XCD's L2
  // holds the grid lists and tables of about one job at a time instead of
  // a slice of every job's.
  const int first_job = (int)(((long)(blockIdx.x & 7) * B.n_jobs) / 8);
  int cur = 0;
  if constexpr (STAGE) {
    // the workgroup's first job, then its table
    if (wib == 0) {
      const int j = pick_job(jobs, B, first_job);
      if (lane == 0) {
        *wg_job = j;
        *wg_t0 = __builtin_amdgcn_s_memrealtime();
      }
    }
    __syncthreads();
    t0 = *wg_t0;
    cur = *wg_job;
    if (cur < 0) return;  // every wave of the workgroup leaves together
    if (!stage_caps(jobs[cur], caps_fill)) caps_lds = nullptr;
    fill_regions<T>(jobs[cur], rows, threadIdx.x, blockDim.x);
    __syncthreads();
  } else if constexpr (!TRACE) {
    cur = pick_job(jobs, B, first_job);
    if (cur < 0) return;
  }
  Packet<T> pk;
  pk.pend = T(0);  // lanes that never get a packet have nothing to credit
  int vx[3] = {0, 0, 0};  // voxel model: the packet's voxel
  pk.state = kDead;

  // outer loop over jobs, inner loop over that job's packets: within the
  // inner loop the job is fixed, so its fields (a noalias read-only kernel
  // argument) and the scene scalars below stay in registers
  for (;;) {
    JobRef a = jobs[cur];
    ScP sc = kptr(a.sc);
    const int nr = sc->n_regions;
    const T delta = Tab<T>::delta(sc);
    const int n_steps = sc->n_steps;
    const int max_steps = sc->max_steps;
    const uint32_t max_events = (uint32_t)sc->max_events;
    bool exhausted = false;     // wave uniform: no packet of this job left to take
    bool resumed_all = false;   // wave uniform: no saved packet of this job left to resume
    int first_surf = 0;         // wave uniform: the lane the interface steps start from

    if constexpr (!STAGE) {
      fill_regions<T>(a, rows, lane, 64);
      wave_fence();
    }
    if constexpr (TRACE) {
      const int id = blockIdx.x * blockDim.x + threadIdx.x;
      exhausted = true;
      if (id < a.n_trace) {
        ln.rec = reinterpret_cast<smcrt_event*>(a.trace_out) + (size_t)id * a.max_records;
        pk.pid = a.trace_ids[id];
        emit<T, TRACE, XF>(a, rg, pk, ln, L);
        if constexpr (GEOM == kGeomVoxel) {
          if (!enter_grid<T, TRACE>(a, rg, pk, vx, ln, L)) pk.state = kDead;
        }
      }
    }

    for (;;) {
      // ---- end of a resident-serving epoch: save the packets in flight
      if constexpr (EPOCH) {
        // (an iteration takes up to 16 steps; a counter of steps between the
        // readings of the clock cost as much as the readings)
        if (!stop && __builtin_amdgcn_s_memrealtime() - t0 > B.deadline) stop = true;
        if (stop) {
          // what this kernel's packets have no use for is saved as constants:
          // held for the save alone, it cost the serving kernels spills and 16
          // requests 8 % of their time
          int at[3] = {0, 0, 0};
          if constexpr (GEOM == kGeomVoxel)
            for (int i = 0; i < 3; ++i) at[i] = vx[i];
          if constexpr (!kRelax) {
            pk.pd = T(-1);
            pk.pl = T(0);
          }
          save_live<T>(B, a, pk.state != kDead, pk, at, lane);
          pk.state = kDead;
          exhausted = true;
          break;
        }
      }

      // ---- refill dead lanes: packets saved by the previous epoch first,
      // then new ids from the job's packet counter
      if constexpr (!TRACE) {
        const bool open = pk.state == kDead && lane < a.lanes;
        const uint64_t dmask = __ballot(open);
        const int ndead = __popcll(dmask);
        if (!exhausted && ndead > 0 && (ndead >= B.refill_min || ndead == a.lanes)) {
          const int leader = __ffsll((unsigned long long)dmask) - 1;
          const int rank = __popcll(dmask & ((1ull << lane) - 1ull));
          int rtake = 0;
          if (EPOCH && a.resume_n > 0 && !resumed_all) {
            unsigned int rb = 0;
            if (lane == leader) rb = atomicAdd(a.resume_next, (unsigned int)ndead);
            rb = __shfl(rb, leader);
            rtake = rb < a.resume_n ? (int)min((unsigned int)ndead, a.resume_n - rb) : 0;
            if (rtake < ndead) resumed_all = true;
            if (open && rank < rtake) {
              int at[3];
              load_saved<T>(a, rb + (unsigned int)rank, pk, at);
              if constexpr (GEOM == kGeomVoxel)
                for (int i = 0; i < 3; ++i) vx[i] = at[i];
            }
          }
          const int rest = ndead - rtake;
          if (rest > 0) {
            unsigned long long base = 0;
            if (lane == leader) base = atomicAdd(a.counter, (unsigned long long)rest);
            base = __shfl(base, leader);
            if (base + (uint64_t)rest >= a.n) exhausted = true;
            if (open && rank >= rtake) {
              const uint64_t id = base + (uint64_t)(rank - rtake);
              if (id < a.n) {
                pk.pid = a.first + id;
                emit<T, TRACE, XF>(a, rg, pk, ln, L);
                if constexpr (GEOM == kGeomVoxel) {
                  if (!enter_grid<T, TRACE>(a, rg, pk, vx, ln, L)) pk.state = kDead;
                }
              }
            }
          }
        }
      }
      const uint64_t lmask = __ballot(pk.state != kDead);
      if (lmask == 0ull) {
        if (exhausted) break;
        continue;
      }

      // ---- moves from voxel to voxel (voxelised model)
      if constexpr (GEOM == kGeomVoxel) {
        voxel_moves<T, TRACE>(a, pk, vx, ln, wt, L, lane, __popcll(lmask), kDueMin, EPOCH ? 16 : INT_MAX, max_steps, max_events);
        if (pk.state == kSurface) pk.state = voxel_face<T, TRACE>(a, rg, pk, vx, ln, L) ? kTransport : kDead;
      }

      // ---- free-flight reuse: the distance evaluated at the last step's
      // start, less the path since, bounds the distance to every surface;
      // an interaction inside that ball (inside a region, so inside the
      // volume) is the one an evaluation would give, so none is made.
      // Margin: delta, plus per reuse 4 units in the last place of the
      // position for the rounding of the moves
      if (GEOM == kGeomSdf && pk.state == kTransport && pk.safe > T(0) && pk.region < nr &&
          pk.links < kReuseLinks) {
        const T s = pk.mut > T(0) ? (T)(pk.tau * (double)pk.inv_mut) : tinf<T>();
        const T pmax = tmax(tabs(pk.p.x), tmax(tabs(pk.p.y), tabs(pk.p.z)));
        const T ulp4 = sizeof(T) == 4 ? T(0x1p-21) : T(0x1p-50);
        if (s <= pk.safe - delta - T(pk.links + 1) * pmax * ulp4) {
          advance(pk, s);
          pk.tau = 0.0;
          pk.state = kInteract;
          pk.safe -= s;
          ++pk.links;
        }
      }

      // ---- sphere-tracing steps (Sec. 2.3), one after the other until
      // kDueMin / 64 of the live lanes are due for the rest of the loop (an
      // interaction or their end), or company has come together at the
      // surfaces: the rest of the loop costs as much for one lane as for all.
      // A wave with few packets left thereby takes step after step without
      // passing through it; the longest packets graze surfaces for thousands
      // of steps, and a short launch lasts as long as they do.  64 runs of
      // 1e5 packets in a batch: as soon as one lane is due 35.2 ms, a quarter
      // 33.2, half 30.4, two thirds 30.3; 1e5 packets of the 50^3 sphere 4.0,
      // 3.9, 3.8, 4.0; 1e7 of the slab 305 all ways.  (The rest of the loop
      // after every step cost the batch 20 % more, the sphere 65 %.)
      uint64_t on = GEOM == kGeomSdf ? __ballot(pk.state == kTransport) : 0ull;
      if (on != 0ull) {
        const ScP hot = fresh(sc);
        const SMCRT_K StepRec<T>* recs = fresh(Tab<T>::steps(a));
        const int nlive = __popcll(lmask);
        int inner = 0;
        uint64_t at;
        do {
          const ScP sc = hot;
          if (pk.state == kTransport) {
            ++pk.steps;
            const bool stall = pk.steps > max_steps || pk.k > max_events;
            T dmin = tinf<T>(), tseg = tinf<T>();
            if (SEG && sc->segment) {
              const T err = Tab<T>::seg_err(sc);
              for (int r = 0; r < nr; ++r) {
                T tb;
                dmin = tmin(dmin, tabs(region_seg<T, XF>(a, r, pk.p, pk.u, err, &tb)));
                tseg = tmin(tseg, tb);
              }
            } else {
              dmin = walk_distance<T, XF>(a, recs, n_steps, pk.p, caps_lds);
            }
            const T om = kRelax ? Tab<T>::relax(sc) : T(1);
            const bool outside = outside_volume<T>(sc, pk.p);
            const T s = pk.mut > T(0) ? (T)(pk.tau * (double)pk.inv_mut) : tinf<T>();
            const bool near = s <= dmin;  // the optical depth runs out before any surface
            // Nearly every step moves dmin on, or s to the interaction.  All
            // that is not such a step goes through one branch: a lone wave
            // takes 30 to 50 cycles for each branch on a vector compare, as
            // long as six dependent instructions
            bool inter = near, move = true, rel = false, jump = false;
            T len = near ? s : dmin;
            if ((SEG && sc->segment) || om > T(1) || stall || outside || (!near && (dmin < delta || pk.region == nr))) {
              bool rejected = false;
              if (om > T(1) && !stall && pk.pl < T(0)) {
                // check of an over-relaxed step (Sec. 5): the open balls of
                // radius pd at its start and dmin at its end hold no surface;
                // unless they cover the step with a margin of delta it goes back
                // to the plain step of pd, and this evaluation is spent
                const T over = -pk.pl;
                if (pk.pd + dmin >= over + delta) {
                  pk.pl = over;
                } else {
                  rejected = true;
                  step_along(pk, pk.pd - over);
                  pk.pl = pk.pd;
                }
              }
              if (stall) {
                atomicAdd(&L.sum[kSStalled], pk.w);
                atomicAdd(&L.cnt[kCStalls], 1ull);
                record<T, TRACE>(a, pk, ln, SMCRT_EV_STALL);
                pk.state = kDead;
                --ln.n_steps;
                move = false;
              } else if (rejected) {
                // the next evaluation starts from the plain step's end
                move = false;
              } else if (outside) {  // outside the simulation volume
                const int face = volume_face<T>(sc, pk.p);
                atomicAdd(&L.sum[kSEscaped + face], pk.w);
                atomicAdd(&L.cnt[kCEscapes], 1ull);
                detect<T>(a, pk, face, Tab<T>::bb_c(sc, face >> 1) + ((face & 1) ? Tab<T>::bb_h(sc, face >> 1) : -Tab<T>::bb_h(sc, face >> 1)));
                record<T, TRACE>(a, pk, ln, SMCRT_EV_ESCAPE);
                pk.state = kDead;
                move = false;
              } else if (!near && dmin < delta) {
                pk.state = kSurface;
                move = false;
              } else {
                // segment tracing: a step may run to the nearest bound along the
                // ray less delta, or delta past the volume's boundary when that
                // comes first
                T seg = dmin;
                if (SEG && sc->segment) {
                  if (!near && tseg - delta > dmin) seg = tmax(dmin, tmin(tseg - delta, volume_exit<T>(sc, pk.p, pk.u) + delta));
                }
                // the packet interacts where its optical depth runs out: within
                // the ball of radius dmin about the step's start, which holds no
                // surface, or (segment tracing) on the free segment ahead, where
                // plain steps would reach it and no free ball about it is known
                inter = near || (SEG && seg > dmin && s <= seg);
                len = inter ? s : dmin;
                if (om > T(1)) {
                  // an over-relaxed step of omega * dmin when it would pass its
                  // check were the surface a plane met at the angle the previous
                  // step saw (its distance falls by (pd - dmin)/pl per unit
                  // length): dmin + dmin - omega (pd - dmin) dmin / pl >= omega
                  // dmin + delta, times pl > 0
                  rel = !inter && pk.pd >= T(0) &&
                        dmin * (Tab<T>::relax_k(sc) * pk.pl - om * (pk.pd - dmin)) >= delta * pk.pl && om * dmin < s;
                  len = rel ? om * dmin : len;
                }
                if (!inter && pk.region == nr) {
                  // ambient skip, when the boxes' margin of delta/2 covers
                  // the rounding of the box test and of the move: 4 units in
                  // the last place of the largest coordinate plus the skip
                  const T tf = ambient_free<T>(sc, nr, pk.p, pk.u, delta);
                  const T pmax = tmax(tabs(pk.p.x), tmax(tabs(pk.p.y), tabs(pk.p.z)));
                  const T ulp4 = sizeof(T) == 4 ? T(0x1p-21) : T(0x1p-50);
                  if (tf > len && tf >= seg && T(0.5) * delta >= ulp4 * (pmax + tf)) {
                    len = tf;
                    jump = true;
                  }
                }
                if (SEG && !inter && !jump && seg > len) {
                  len = seg;
                  jump = true;
                  rel = false;
                }
              }
            }
            ++ln.n_steps;
            pk.safe = near && move && pk.region < nr ? dmin - s : T(-1);
            if (move) {
              advance(pk, len);
              const double left = pk.tau - (double)pk.mut * (double)len;
              pk.tau = inter ? 0.0 : left;
              pk.state = inter ? kInteract : kTransport;
              pk.links = near ? 0 : pk.links;
              if constexpr (kRelax) {
                pk.pd = inter ? pk.pd : (jump ? T(-1) : dmin);
                pk.pl = inter ? pk.pl : (rel && !jump ? -len : len);
              }
            }
          }
          on = __ballot(pk.state == kTransport);
          if (on == lmask) continue;
          at = __ballot(pk.state == kSurface);
          if (on == 0ull || __popcll(lmask & ~(on | at)) * 64 >= kDueMin * nlive ||
              __popcll(at) * 64 >= B.surface_min * nlive)
            break;
          // (resident serving: back to the deadline every 16 steps)
        } while (!EPOCH || ++inner < 16);
      }

      // ---- interface steps, gathered: up to eight packets an iteration,
      // taken from a lane that moves on with the iterations, so that none
      // waits behind the others for good
      int hit = -1;  // the packet's interface slot
      if constexpr (GEOM == kGeomSdf) {
        const bool at = pk.state == kSurface;
        const uint64_t smask = __ballot(at);
        const int nsurf = __popcll(smask);
        if (nsurf > 0 && nsurf * 64 >= B.surface_min * __popcll(lmask)) {
          first_surf = (first_surf + 8) & 63;
          const uint64_t turned = (smask >> first_surf) | (smask << ((64 - first_surf) & 63));
          const int rank = __popcll(turned & ((1ull << ((lane - first_surf) & 63)) - 1ull));
          SurfaceSlot* S = Hw[wib];
          if (at && rank < kSurfaceSlots) {
            SurfaceSlot& s = S[rank];
            V3<double> p = to_d(pk.p);
            if constexpr (sizeof(T) == 4) p = p + to_d(pk.pe);  // the position's compensated sum
            const V3<double> u = to_d(pk.u);
            s.p[0] = p.x; s.p[1] = p.y; s.p[2] = p.z;
            s.u[0] = u.x; s.u[1] = u.y; s.u[2] = u.z;
            s.region = pk.region;
          }
          wave_fence();
          surface_geometry<XF>(a, S, nsurf < kSurfaceSlots ? nsurf : kSurfaceSlots, lane);
          if (at && rank < kSurfaceSlots && surface_arrive<T>(a, rg, S[rank], pk, L)) hit = rank;
        }
      }

      // ---- tally: lanes whose packet ended, is about to scatter or stands
      // on an interface (its position jumps or its direction changes next)
      // credit their straight path since the last event to the grid, together
      if constexpr (GEOM == kGeomSdf) {
        const bool due = pk.pend > T(0) && (pk.state >= kInteract || hit >= 0);
        tally_path<T>(a, pk, due, ln, wt);
        if (due) pk.pend = T(0);
        if (hit >= 0) {
          pk.pend = T(0);
          surface_event<T, TRACE>(a, rg, Hw[wib][hit], pk, ln, L);
        }
      }

      // ---- interactions
      if (pk.state == kInteract) {
        pk.state = kTransport;
        if (!interact<T, TRACE>(a, rg, pk, ln, L)) pk.state = kDead;
      }

      // ---- grid additions staged this iteration, as full-wave atomics.
      // Last in the iteration: one counter tracks a wave's vector loads and
      // its atomics in issue order, so the first per-lane table load after
      // a drain (the region's coefficients in the interaction) waits until
      // every drained atomic has completed at the L2.  Issued here, they
      // complete while the next iteration's step runs.
      if (a.fluence != nullptr) {
        tally_drain(a.fluence, *ln.stage, wt, kDrain, lane);
      }
    }

    if constexpr (TRACE) {
      const int id = blockIdx.x * blockDim.x + threadIdx.x;
      if (id < a.n_trace) a.trace_count[id] = ln.n_rec < a.max_records ? ln.n_rec : a.max_records;
      flush_wave(a, ln, wt, L, lane);
      break;
    } else if constexpr (STAGE) {
      // job drained by this wave: hand in its sums; once every wave is done
      // with the job (and its table), the workgroup takes the next one
      flush_wave(a, ln, wt, L, lane);
      __syncthreads();
      if (wib == 0) {
        const bool late = EPOCH && __builtin_amdgcn_s_memrealtime() - t0 > B.deadline;
        const int j = late ? -1 : pick_job(jobs, B, cur + 1);
        if (lane == 0) *wg_job = j;
      }
      __syncthreads();
      cur = *wg_job;
      if (cur < 0) break;
      caps_lds = (LdsCaps)caps_fill;
      if (!stage_caps(jobs[cur], caps_fill)) caps_lds = nullptr;
      fill_regions<T>(jobs[cur], rows, threadIdx.x, blockDim.x);
      __syncthreads();
    } else {
      // job drained by this wave (or the epoch ended): hand in its sums,
      // take the next job
      flush_wave(a, ln, wt, L, lane);
      if (stop) break;
      cur = pick_job(jobs, B, cur + 1);
      if (cur < 0) break;
    }
  }
}

__global__ void zero_u64_kernel(unsigned long long* p) { *p = 0ull; }

__global__ void scale_kernel(const double* __restrict__ in, double* __restrict__ out, size_t n, double s) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    out[i] = in[i] * s;
}

template <int GEOM, bool XF, bool SEG = false>
static void launch_geom(int precision, bool trace, dim3 grid, dim3 block, const BatchArgs& args, hipStream_t stream) {
  const bool epoch = args.deadline != 0;
  if (precision == 1) {
    if (trace) hipLaunchKernelGGL((walk_kernel<double, true, GEOM, XF, false, false, SEG>), grid, block, 0, stream, args.jobs, args);
    else if (epoch) hipLaunchKernelGGL((walk_kernel<double, false, GEOM, XF, false, true, SEG>), grid, block, 0, stream, args.jobs, args);
    else hipLaunchKernelGGL((walk_kernel<double, false, GEOM, XF, false, false, SEG>), grid, block, 0, stream, args.jobs, args);
  } else {
    if (trace) hipLaunchKernelGGL((walk_kernel<float, true, GEOM, XF, false, false, SEG>), grid, block, 0, stream, args.jobs, args);
    else if (epoch) hipLaunchKernelGGL((walk_kernel<float, false, GEOM, XF, false, true, SEG>), grid, block, 0, stream, args.jobs, args);
    else hipLaunchKernelGGL((walk_kernel<float, false, GEOM, XF, false, false, SEG>), grid, block, 0, stream, args.jobs, args);
  }
}

// args.geometry is the launch class: the geometry model plus kLaunchXf when
// the jobs' scenes have placed or modified primitives
hipError_t launch_walk(int precision, bool trace, const LaunchCfg& cfg, const BatchArgs& args, hipStream_t stream) {
  if (!args.jobs || args.n_jobs < 1 || (trace && args.n_jobs != 1)) return hipErrorInvalidValue;
  if (args.refill_min < 1 || args.refill_min > 64 || args.surface_min < 1 || args.surface_min > 64) return hipErrorInvalidValue;
  if (args.geometry < 0 || args.geometry >= kLaunchClasses) return hipErrorInvalidValue;
  if (args.geometry == kLaunchStaged) {
    // FP32 staged-capsule walk: workgroups of 16 waves, no trace variant
    if (precision != 0 || trace || cfg.block != 1024 || cfg.grid < 1) return hipErrorInvalidConfiguration;
    if (args.deadline)
      hipLaunchKernelGGL((walk_kernel<float, false, kGeomSdf, false, true, true, false>), dim3(cfg.grid), dim3(1024), 0, stream,
                         args.jobs, args);
    else
      hipLaunchKernelGGL((walk_kernel<float, false, kGeomSdf, false, true, false, false>), dim3(cfg.grid), dim3(1024), 0, stream,
                         args.jobs, args);
    return hipGetLastError();
  }
  if (cfg.block < 64 || cfg.block > 256 || cfg.block % 64 || cfg.grid < 1) return hipErrorInvalidConfiguration;
  dim3 grid(cfg.grid), block(cfg.block);
  switch (args.geometry) {
    case kGeomSdf: launch_geom<kGeomSdf, false>(precision, trace, grid, block, args, stream); break;
    case kGeomVoxel: launch_geom<kGeomVoxel, false>(precision, trace, grid, block, args, stream); break;
    case kGeomSdf + kLaunchXf: launch_geom<kGeomSdf, true>(precision, trace, grid, block, args, stream); break;
    case kLaunchSegment: launch_geom<kGeomSdf, false, true>(precision, trace, grid, block, args, stream); break;
    default: launch_geom<kGeomVoxel, true>(precision, trace, grid, block, args, stream); break;
  }
  return hipGetLastError();
}

__global__ void zero_u64_n_kernel(unsigned long long* p, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0ull;
}

hipError_t launch_zero_u64_n(unsigned long long* p, int n, hipStream_t stream) {
  if (!p || n < 1) return hipErrorInvalidValue;
  const int blocks = (n + 255) / 256;
  hipLaunchKernelGGL(zero_u64_n_kernel, dim3(blocks < 1024 ? blocks : 1024), dim3(256), 0, stream, p, n);
  return hipGetLastError();
}

__global__ void zero_f64_kernel(double* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0.0;
}

// F (x fastest, nx*ny*nz) += S (2x2x2 bricks)
__global__ void brick_add_kernel(const double* __restrict__ S, double* __restrict__ F, int nx, int ny, int nz) {
  const size_t n = (size_t)nx * ny * nz;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int x = (int)(i % (size_t)nx), y = (int)((i / (size_t)nx) % (size_t)ny), z = (int)(i / ((size_t)nx * ny));
    F[i] += S[brick_index(x, y, z, nx, ny)];
  }
}

hipError_t launch_zero_f64(double* p, size_t n, hipStream_t stream) {
  if (!p || n == 0) return hipErrorInvalidValue;
  const size_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(zero_f64_kernel, dim3(blocks < 4096 ? (unsigned)blocks : 4096u), dim3(256), 0, stream, p, n);
  return hipGetLastError();
}

hipError_t launch_brick_add(const double* S, double* F, int nx, int ny, int nz, hipStream_t stream) {
  if (!S || !F || nx < 1 || ny < 1 || nz < 1) return hipErrorInvalidValue;
  const size_t n = (size_t)nx * ny * nz, blocks = (n + 255) / 256;
  hipLaunchKernelGGL(brick_add_kernel, dim3(blocks < 4096 ? (unsigned)blocks : 4096u), dim3(256), 0, stream, S, F, nx, ny, nz);
  return hipGetLastError();
}

hipError_t launch_zero_u64(unsigned long long* p, hipStream_t stream) {
  hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(1), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_scale(const double* in, double* out, size_t n, double scale, hipStream_t stream) {
  size_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(scale_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, in, out, n, scale);
  return hipGetLastError();
}

template <int GEOM, bool XF, bool SEG = false>
static hipError_t occupancy(int* n, int precision, int block) {
  return precision == 1
             ? hipOccupancyMaxActiveBlocksPerMultiprocessor(n, walk_kernel<double, false, GEOM, XF, false, false, SEG>, block, 0)
             : hipOccupancyMaxActiveBlocksPerMultiprocessor(n, walk_kernel<float, false, GEOM, XF, false, false, SEG>, block, 0);
}

int walk_max_blocks_per_cu(int precision, int block, int launch_class) {
  int n = 0;
  hipError_t e;
  if (launch_class == kLaunchStaged) {
    if (precision != 0 || block != 1024) return 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, walk_kernel<float, false, kGeomSdf, false, true, false, false>, 1024, 0);
    return e == hipSuccess ? n : 0;
  }
  switch (launch_class) {
    case kGeomSdf: e = occupancy<kGeomSdf, false>(&n, precision, block); break;
    case kGeomVoxel: e = occupancy<kGeomVoxel, false>(&n, precision, block); break;
    case kGeomSdf + kLaunchXf: e = occupancy<kGeomSdf, true>(&n, precision, block); break;
    case kLaunchSegment: e = occupancy<kGeomSdf, false, true>(&n, precision, block); break;
    default: e = occupancy<kGeomVoxel, true>(&n, precision, block); break;
  }
  return e == hipSuccess ? n : 0;
}

}  // namespace smcrt