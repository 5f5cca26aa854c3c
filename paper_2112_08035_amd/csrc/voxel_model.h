// voxel_model.h -- device functions of the voxelised-geometry model, the
// comparison model of Sec. 3: the scene is replaced by the region of each
// fluence-grid voxel centre (voxelize_kernel in voxel.hip), and a packet
// moves from voxel face to voxel face.  Emission, interactions, the random
// stream and the tallies are the SDF walk's own (walk_common.h); only the
// geometry differs:
//   - beyond the grid lies the ambient medium; a packet born outside the
//     grid travels to it unattenuated and untallied, or escapes if it misses;
//   - a face between voxels of equal refractive index is crossed without an
//     event (the region, hence mu_a and mu_s, may still change there);
//   - a face where the index changes, the grid faces included, is an
//     interface event with the axis as normal: Fresnel in FP64, reflection
//     or vector Snell refraction, next event index, variate word 0;
//   - transmission through a grid face is an escape through that face.
#pragma once
#include "walk_common.h"

namespace smcrt {

__device__ __forceinline__ int vox_index(ScP sc, const int v[3]) {
  return v[0] + sc->g_dims[0] * (v[1] + sc->g_dims[1] * v[2]);
}

template <typename T>
__device__ __forceinline__ T comp(const V3<T>& a, int i) {
  return i == 0 ? a.x : (i == 1 ? a.y : a.z);
}
template <typename T>
__device__ __forceinline__ void set_comp(V3<T>& a, int i, T x) {
  if (i == 0) a.x = x;
  else if (i == 1) a.y = x;
  else a.z = x;
}

// escape through grid face `face`; on_grid: the packet is on that face (it
// reached the grid), so it is seen by the escape image
template <typename T, bool TRACE>
__device__ __forceinline__ void escape_face(JobRef a, Packet<T>& pk, Lane& ln, LdsTallies& L, int face, bool on_grid) {
  ScP sc = kptr(a.sc);
  pk.region = sc->n_regions;
  atomicAdd(&L.sum[kSEscaped + face], pk.w);
  atomicAdd(&L.cnt[kCEscapes], 1ull);
  if (on_grid) detect<T>(a, pk, face, (face & 1) ? Tab<T>::g_hi(sc, face >> 1) : Tab<T>::g_lo(sc, face >> 1));
  record<T, TRACE>(a, pk, ln, SMCRT_EV_ESCAPE);
}

// Interface event at the face of axis ax between the packet's medium and
// region r2 (n_regions = ambient).  FP64 Fresnel with the axis as normal.
// Returns true when the packet passed into r2, false when it reflected.
template <typename T, bool TRACE>
__device__ bool voxel_interface(JobRef a, Regions<T> rg, Packet<T>& pk, Lane& ln, LdsTallies& L, int ax, int r2, double n1,
                                double n2) {
  pk.k += 1;
  pk.steps = 0;
  atomicAdd(&L.cnt[kCInterfaces], 1ull);
  const U4 rr = philox10(pk.k, (uint32_t)pk.pid, (uint32_t)(pk.pid >> 32), 0u, (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
  const double x0 = xi_of<double>(rr.w0);
  V3<double> u = to_d(pk.u);
  const double ua = comp(u, ax);
  const double ci = __builtin_fabs(ua);
  double ct;
  const double R = fresnel(n1, n2, ci, &ct);
  if (x0 < R) {  // specular reflection: the axis component flips
    set_comp(pk.u, ax, -comp(pk.u, ax));
    atomicAdd(&L.cnt[kCReflections], 1ull);
    record<T, TRACE>(a, pk, ln, SMCRT_EV_REFLECT);
    return false;
  }
  const double eta = n1 / n2, sg = ua > 0.0 ? 1.0 : -1.0;
  u = eta * u;
  set_comp(u, ax, comp(u, ax) + (ct - eta * ci) * sg);
  u = (1.0 / __builtin_sqrt(dot(u, u))) * u;
  pk.u = from_d<T>(u);
  set_region(rg, pk, r2);
  atomicAdd(&L.cnt[kCRefractions], 1ull);
  record<T, TRACE>(a, pk, ln, SMCRT_EV_REFRACT);
  return true;
}

// After emission: place the packet in its voxel v, entering the grid from
// outside if it was born there.  Returns false when the packet has ended
// (it missed the grid, or reflected off the grid face it arrived at).
template <typename T, bool TRACE>
__device__ bool enter_grid(JobRef a, Regions<T> rg, Packet<T>& pk, int v[3], Lane& ln, LdsTallies& L) {
  ScP sc = kptr(a.sc);
  const int nr = sc->n_regions;
  const V3<T> p = pk.p, u = pk.u;
  bool inside = true;
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (comp(p, i) < Tab<T>::g_lo(sc, i) || comp(p, i) > Tab<T>::g_hi(sc, i)) inside = false;
  int entry = -1;
  if (!inside) {  // slab test against the grid box
    T t0 = T(0), t1 = tinf<T>();
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const T pi = comp(p, i), ui = comp(u, i), lo = Tab<T>::g_lo(sc, i), hi = Tab<T>::g_hi(sc, i);
      if (ui == T(0)) {
        if (pi < lo || pi > hi) t1 = T(-1);
      } else {
        const T ta = (lo - pi) / ui, tb = (hi - pi) / ui;
        const T tn = tmin(ta, tb), tx = tmax(ta, tb);
        if (tn > t0) {
          t0 = tn;
          entry = i;
        }
        t1 = tmin(t1, tx);
      }
    }
    if (!(t1 > t0) || entry < 0) {  // misses the grid: out through the nearest box face
      int face = 0;
      T best = -tinf<T>();
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const T lo = Tab<T>::g_lo(sc, i), hi = Tab<T>::g_hi(sc, i);
        const T c = T(0.5) * (lo + hi), e = tabs(comp(p, i) - c) - T(0.5) * (hi - lo);
        if (e > best) {
          best = e;
          face = 2 * i + (comp(p, i) > c ? 1 : 0);
        }
      }
      escape_face<T, TRACE>(a, pk, ln, L, face, false);
      return false;
    }
    shift(pk, t0);
    set_region(rg, pk, nr);  // in the ambient medium, on the grid face
  }
  // voxel holding the point; on a voxel face, the one the packet moves into
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int n = sc->g_dims[i];
    const T x = (comp(pk.p, i) - Tab<T>::g_lo(sc, i)) / Tab<T>::g_d(sc, i);
    const T fl = floor(x);
    int k = (int)tclamp(fl, T(-1), T(n));
    if (comp(u, i) < T(0) && x == fl) k -= 1;
    if (i == entry) k = comp(u, i) > T(0) ? 0 : n - 1;
    v[i] = k < 0 ? 0 : (k >= n ? n - 1 : k);
  }
  const int r2 = a.vox[vox_index(sc, v)];
  if (entry < 0) {
    set_region(rg, pk, r2);
    return true;
  }
  const double n1 = rg[nr].n, n2 = rg[r2].n;
  if (n1 == n2) {
    set_region(rg, pk, r2);
    return true;
  }
  if (voxel_interface<T, TRACE>(a, rg, pk, ln, L, entry, r2, n1, n2)) return true;
  // reflected off the grid: it leaves through the face it came to
  escape_face<T, TRACE>(a, pk, ln, L, 2 * entry + (comp(pk.u, entry) > T(0) ? 1 : 0), true);
  return false;
}

// The way to the next face of one axis (hi: the upper one), from the
// compensated position (FP32: p + pe): the gap by u, y = 1 / u, as corrections
// of the product by its residual (Markstein), the last steps of a division
// without its own reciprocal.  Infinite along the axis's planes (u = 0), and
// where the product is: from there on the residual overflows, and no scene is
// as large.  (FP32: a gap under 2^-102 has a residual that underflows, and a
// quotient that may be 1 ulp off; a |u| under 2^-128 has no reciprocal and
// crosses only the faces it stands on.)
template <typename T>
__device__ __forceinline__ T face_way(T lo, T d, int v, bool hi, T p, T pe, T u, T y) {
  constexpr T kFar = sizeof(T) == 4 ? T(0x1p100) : T(0x1p1000);
  const T face = lo + T(v + (hi ? 1 : 0)) * d;
  const T x = (face - p) - pe, q0 = x * y;
  T q = tfma(tfma(-u, q0, x), y, q0);
  q = tfma(tfma(-u, q, x), y, q);
  return u == T(0) || q0 >= kFar ? tinf<T>() : tmax(q, T(0));  // (behind the face by rounding: 0)
}

// Moves of the voxel walk, one after the other until kDueMin / 64 of the live
// lanes are due for the rest of the loop: each to the exit face of the
// packet's voxel v or to the interaction point (pk.state = kInteract),
// whichever is nearer, tallying the piece.  A face where the region changes
// or the grid ends is left to voxel_face (pk.state = kSurface, the face in
// pk.links).  At most `most` moves.  Called with every lane of the wave active.
//
// What bounds it is the chain of one move -- three divisions, the region of
// the next voxel from memory, the tally -- and, with the card full, their
// instructions.  So the reciprocals are kept for as long as the direction is,
// the next voxel's region is asked for before the piece is tallied, and
// the tally is the SDF walk's, with no lane-by-lane staging.  1e6 packets of
// the voxelised cylinder (256^3) 45.0 to 36.7 ms, 1e5 15.5 to 10.9, a lone
// packet's move 1.31 to 0.85 us.  (A fifth wave per SIMD: no faster; bricks
// for its tally: 38.1 against 37.6; true divisions where a component is small,
// behind a branch or in a loop of their own, 1 and 2 % slower.)
template <typename T, bool TRACE>
__device__ __forceinline__ void voxel_moves(JobRef a, Packet<T>& pk, int v[3], Lane& ln, WaveTally& wt, LdsTallies& L,
                                            int lane, int n_live, int due_min, int most, int max_steps,
                                            uint32_t max_events) {
  uint64_t on = __ballot(pk.state == kTransport);
  if (on == 0ull) return;
  ScP sc = fresh(kptr(a.sc));
  const int nx = sc->g_dims[0], ny = sc->g_dims[1], nz = sc->g_dims[2];
  const V3<T> u = pk.u, y = mk(T(1) / u.x, T(1) / u.y, T(1) / u.z);
  const bool ux = u.x > T(0), uy = u.y > T(0), uz = u.z > T(0);
  int idx = vox_index(sc, v);
  do {
    bool go = pk.state == kTransport;
    if (go) {
      if (++pk.steps > max_steps || pk.k > max_events) {
        atomicAdd(&L.sum[kSStalled], pk.w);
        atomicAdd(&L.cnt[kCStalls], 1ull);
        record<T, TRACE>(a, pk, ln, SMCRT_EV_STALL);
        pk.state = kDead;
        go = false;
      }
    }
    T len = T(0);
    int r2 = -1, face = 0, step = 0, dir = 0;
    bool inter = false;
    if (go) {
      ++ln.n_steps;
      const T tx = face_way(Tab<T>::g_lo(sc, 0), Tab<T>::g_d(sc, 0), v[0], ux, pk.p.x, pk.pe.x, u.x, y.x);
      const T ty = face_way(Tab<T>::g_lo(sc, 1), Tab<T>::g_d(sc, 1), v[1], uy, pk.p.y, pk.pe.y, u.y, y.y);
      const T tz = face_way(Tab<T>::g_lo(sc, 2), Tab<T>::g_d(sc, 2), v[2], uz, pk.p.z, pk.pe.z, u.z, y.z);
      const bool bx = tx <= ty && tx <= tz, by = !bx && ty <= tz;  // (ties: x before y before z)
      const T texit = bx ? tx : (by ? ty : tz);
      const bool up = bx ? ux : (by ? uy : uz);
      const int va = bx ? v[0] : (by ? v[1] : v[2]), na = bx ? nx : (by ? ny : nz);
      dir = up ? 1 : -1;
      face = (bx ? 0 : (by ? 2 : 4)) + (up ? 1 : 0);
      step = (bx ? 1 : (by ? nx : nx * ny)) * dir;
      if (va != (up ? na - 1 : 0)) r2 = (int)a.vox[idx + step];
      const T s = pk.mut > T(0) ? (T)(pk.tau * (double)pk.inv_mut) : tinf<T>();
      inter = s <= texit;
      len = inter ? s : texit;
      shift(pk, len);
      pk.tau = inter ? 0.0 : pk.tau - (double)pk.mut * (double)len;
    }
    if (a.fluence != nullptr) {
      run_piece<true>(a.fluence, *ln.stage, wt, ln.run, go && len > T(0), idx, pk.w * (double)len);
      tally_drain(a.fluence, *ln.stage, wt, kDrain, lane);
    }
    if (go) {
      const bool stay = !inter && r2 == pk.region;
      idx += stay ? step : 0;
      v[0] += stay && face < 2 ? dir : 0;
      v[1] += stay && (face >> 1) == 1 ? dir : 0;
      v[2] += stay && face >= 4 ? dir : 0;
      pk.links = face;
      pk.state = inter ? kInteract : (stay ? kTransport : kSurface);
    }
    on = __ballot(pk.state == kTransport);
  } while (on != 0ull && (n_live - __popcll(on)) * 64 < due_min * n_live && --most > 0);
}

// A packet on face pk.links of its voxel v, where the region changes or the
// grid ends.  Returns false when the packet has ended (escape).
template <typename T, bool TRACE>
__device__ bool voxel_face(JobRef a, Regions<T> rg, Packet<T>& pk, int v[3], Lane& ln, LdsTallies& L) {
  ScP sc = kptr(a.sc);
  const int face = pk.links, ax = face >> 1;
  int w2[3] = {v[0], v[1], v[2]};
  w2[ax] += (face & 1) ? 1 : -1;
  const bool off = w2[ax] < 0 || w2[ax] >= sc->g_dims[ax];
  const int r2 = off ? sc->n_regions : (int)a.vox[vox_index(sc, w2)];
  const double n1 = rg[pk.region].n, n2 = rg[r2].n;
  if (n1 == n2) {
    if (off) {
      escape_face<T, TRACE>(a, pk, ln, L, face, true);
      return false;
    }
    v[0] = w2[0]; v[1] = w2[1]; v[2] = w2[2];
    if (r2 != pk.region) set_region(rg, pk, r2);
    return true;
  }
  if (!voxel_interface<T, TRACE>(a, rg, pk, ln, L, ax, r2, n1, n2)) return true;  // reflected: same voxel
  if (off) {  // transmitted out of the grid
    atomicAdd(&L.sum[kSEscaped + face], pk.w);
    atomicAdd(&L.cnt[kCEscapes], 1ull);
    detect<T>(a, pk, face, (face & 1) ? Tab<T>::g_hi(sc, face >> 1) : Tab<T>::g_lo(sc, face >> 1));
    record<T, TRACE>(a, pk, ln, SMCRT_EV_ESCAPE);
    return false;
  }
  v[0] = w2[0]; v[1] = w2[1]; v[2] = w2[2];
  return true;
}

}  // namespace smcrt
