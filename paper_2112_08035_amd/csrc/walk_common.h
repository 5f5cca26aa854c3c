// walk_common.h -- device code shared by the SDF walk (walk.hip) and the
// voxel-model walk (voxel.hip): vector types, the Philox stream, scene
// table access, the region SDFs, the path-length tally, the packet state,
// emission, interactions, and the wave-level job picking and flushing.
#pragma once
#include <hip/hip_runtime.h>

#include "../../include/smcrt.h"
#include "layout.h"

namespace smcrt {

// Scene tables, primitives, uniform grids and job tables are read-only for a
// kernel's lifetime: they are read through the constant address space, so
// wave-uniform reads become scalar loads into SGPRs and per-lane reads plain
// global loads.  The fluence grid is written through the global space.
#define SMCRT_K __attribute__((address_space(4)))
#define SMCRT_G __attribute__((address_space(1)))
using ScP = const SMCRT_K SceneHeader*;
using RegRef = const SMCRT_K Region&;
using JobRef = const SMCRT_K WalkArgs&;
template <class X>
__device__ __forceinline__ const SMCRT_K X* kptr(const X* p) {
  return (const SMCRT_K X*)p;
}

// The same pointer, opaque to the compiler.  Table values read through it are
// read where they are used: read through the plain pointer, the compiler moves
// the loads of all of them to the start of the job, runs out of scalar
// registers and fetches them back from vector lanes one by one.
template <class X>
__device__ __forceinline__ const SMCRT_K X* fresh(const SMCRT_K X* p) {
  uint64_t v = (uint64_t)p;
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+s"(v));
#endif
  return (const SMCRT_K X*)v;
}

// Ends an expression: the compiler fuses no multiplication and addition
// across it, so what is computed on either side rounds the same wherever the
// code is inlined.
template <typename T>
__device__ __forceinline__ void hold(T& x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(x));
#endif
}

// ------------------------------------------------------------------ types

template <typename T>
struct V3 {
  T x, y, z;
};
template <typename T>
__device__ __forceinline__ V3<T> mk(T x, T y, T z) { return V3<T>{x, y, z}; }
template <typename T>
__device__ __forceinline__ V3<T> operator+(V3<T> a, V3<T> b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
template <typename T>
__device__ __forceinline__ V3<T> operator-(V3<T> a, V3<T> b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
template <typename T>
__device__ __forceinline__ V3<T> operator*(T s, V3<T> a) { return {s * a.x, s * a.y, s * a.z}; }
template <typename T>
__device__ __forceinline__ T dot(V3<T> a, V3<T> b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
template <typename T>
__device__ __forceinline__ V3<double> to_d(V3<T> a) { return {(double)a.x, (double)a.y, (double)a.z}; }
template <typename T>
__device__ __forceinline__ V3<T> from_d(V3<double> a) { return {(T)a.x, (T)a.y, (T)a.z}; }

// Correctly rounded, as sqrtf is, by the steps the compiler takes for it on
// this target: the instruction's result (1 ulp) or a neighbour, by the signs
// of the residuals, from an operand scaled up where its residual would
// underflow.  sqrtf also picks out 0 and infinity, which here come through the
// comparisons as they are.  14 instructions for 16, on the chain of every
// step: 1e6 packets of the reflectance image 20.1 to 19.7 ms, 1e3 of the 50^3
// sphere 1.06 to 1.04.  (Without the scaling 19.3 and 1.03 ms, but denormal
// operands, of lengths under 1e-19, gave nearly zero.)
__device__ __forceinline__ float tsqrt(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  const bool small = x < 0x1p-96f;
  x = __builtin_ldexpf(x, small ? 64 : 0);
  const float s = __builtin_amdgcn_sqrtf(x);
  const float lo = __builtin_bit_cast(float, __builtin_bit_cast(int, s) - 1);
  const float hi = __builtin_bit_cast(float, __builtin_bit_cast(int, s) + 1);
  const float q = __builtin_fmaf(-lo, s, x) <= 0.0f ? lo : s;
  const float r = __builtin_fmaf(-hi, s, x) > 0.0f ? hi : q;
  return __builtin_ldexpf(r, small ? -32 : 0);
#else
  return __builtin_sqrtf(x);
#endif
}
__device__ __forceinline__ double tsqrt(double x) { return __builtin_sqrt(x); }
__device__ __forceinline__ float tlog(float x) { return __logf(x); }
__device__ __forceinline__ double tlog(double x) { return log(x); }
__device__ __forceinline__ void tsincos_2pi(float xi, float* s, float* c) {
  float a = 6.2831853071795864769f * xi;
  *s = __sinf(a);
  *c = __cosf(a);
}
__device__ __forceinline__ void tsincos_2pi(double xi, double* s, double* c) { sincos(2.0 * M_PI * xi, s, c); }
__device__ __forceinline__ float tdiv(float a, float b) { return __fdividef(a, b); }
__device__ __forceinline__ double tdiv(double a, double b) { return a / b; }
// min, max, abs and clamp as single instructions (v_min/v_max, an abs
// source modifier, v_med3 for a clamp); a NaN operand yields the other one
template <typename T>
__device__ __forceinline__ T tmin(T a, T b) {
  if constexpr (sizeof(T) == 4) return __builtin_fminf(a, b);
  else return __builtin_fmin(a, b);
}
template <typename T>
__device__ __forceinline__ T tmax(T a, T b) {
  if constexpr (sizeof(T) == 4) return __builtin_fmaxf(a, b);
  else return __builtin_fmax(a, b);
}
template <typename T>
__device__ __forceinline__ T tabs(T a) {
  if constexpr (sizeof(T) == 4) return __builtin_fabsf(a);
  else return __builtin_fabs(a);
}
template <typename T>
__device__ __forceinline__ T tfma(T a, T b, T c) {
  if constexpr (sizeof(T) == 4) return __builtin_fmaf(a, b, c);
  else return __builtin_fma(a, b, c);
}
// dot() with its roundings fixed: the same wherever it is inlined
template <typename T>
__device__ __forceinline__ T fdot(V3<T> a, V3<T> b) {
  return tfma(a.z, b.z, tfma(a.x, b.x, a.y * b.y));
}
// p - t e, and x^2 + y^2, their roundings fixed too
template <typename T>
__device__ __forceinline__ V3<T> fback(V3<T> p, T t, V3<T> e) {
  return {tfma(-t, e.x, p.x), tfma(-t, e.y, p.y), tfma(-t, e.z, p.z)};
}
template <typename T>
__device__ __forceinline__ T sum_sq(T x, T y) { return tfma(x, x, y * y); }
template <typename T>
__device__ __forceinline__ T tclamp(T x, T lo, T hi) { return tmin(tmax(x, lo), hi); }
template <typename T>
__device__ __forceinline__ T tinf();
template <>
__device__ __forceinline__ float tinf<float>() { return __builtin_inff(); }
template <>
__device__ __forceinline__ double tinf<double>() { return __builtin_inf(); }

// ------------------------------------------------------------------ Philox

// Philox4x32-10 (Salmon et al., SC'11): ten rounds; each multiplies words 0
// and 2 by the round constants, swaps in the high halves xor-ed with the
// other words and the round key, and bumps the key by the Weyl constants.
struct U4 {
  uint32_t w0, w1, w2, w3;
};
__device__ __forceinline__ U4 philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t m0 = (uint64_t)0xD2511F53u * (uint64_t)c0;
    const uint64_t m1 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
    const uint32_t x0 = (uint32_t)(m1 >> 32) ^ c1 ^ k0;
    const uint32_t x2 = (uint32_t)(m0 >> 32) ^ c3 ^ k1;
    c1 = (uint32_t)m1;
    c3 = (uint32_t)m0;
    c0 = x0;
    c2 = x2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return U4{c0, c1, c2, c3};
}

// a 32-bit word -> (m + 1/2) / 2^23 with m its top 23 bits; exact in FP32
template <typename T>
__device__ __forceinline__ T xi_of(uint32_t w) {
  return ((T)(w >> 9) + T(0.5)) * T(1.0 / 8388608.0);
}

// ------------------------------------------------------------------ scene

// the capsule table a staged-capsule workgroup holds in LDS (two float4 per
// capsule: a.x a.y a.z ba.x | ba.y ba.z 1/|ba|^2 r)
typedef float F4 __attribute__((ext_vector_type(4)));
using LdsCaps = const __attribute__((address_space(3))) F4*;

template <typename T>
struct Tab;
template <>
struct Tab<float> {
  static __device__ __forceinline__ const SMCRT_K PrimF* prims(JobRef a) { return kptr(a.pf); }
  static __device__ __forceinline__ const SMCRT_K float* caps(JobRef a) { return kptr(a.acc_capf); }
  static __device__ __forceinline__ const SMCRT_K StepRec<float>* steps(JobRef a) { return kptr(a.step_f); }
  static __device__ __forceinline__ float hg_b(RegRef r) { return r.hg_bf; }
  static __device__ __forceinline__ float hg_c(RegRef r) { return r.hg_cf; }
  static __device__ __forceinline__ float hg_d(RegRef r) { return r.hg_df; }
  static __device__ __forceinline__ float k(RegRef r) { return r.kf; }
  static __device__ __forceinline__ float inv_k(RegRef r) { return r.inv_kf; }
  static __device__ __forceinline__ float mut(RegRef r) { return r.mutf; }
  static __device__ __forceinline__ float inv_mut(RegRef r) { return r.inv_mutf; }
  static __device__ __forceinline__ V3<float> bb_c(ScP s) { return {s->bb_cf[0], s->bb_cf[1], s->bb_cf[2]}; }
  static __device__ __forceinline__ V3<float> bb_h(ScP s) { return {s->bb_hf[0], s->bb_hf[1], s->bb_hf[2]}; }
  static __device__ __forceinline__ float bb_c(ScP s, int i) { return s->bb_cf[i]; }
  static __device__ __forceinline__ float bb_h(ScP s, int i) { return s->bb_hf[i]; }
  static __device__ __forceinline__ V3<float> g_lo(ScP s) { return {s->g_lof[0], s->g_lof[1], s->g_lof[2]}; }
  static __device__ __forceinline__ V3<float> g_inv(ScP s) { return {s->g_inv_df[0], s->g_inv_df[1], s->g_inv_df[2]}; }
  static __device__ __forceinline__ float g_d(ScP s, int i) { return s->g_df[i]; }
  static __device__ __forceinline__ float g_lo(ScP s, int i) { return s->g_lof[i]; }
  static __device__ __forceinline__ float g_hi(ScP s, int i) { return s->g_hif[i]; }
  static __device__ __forceinline__ float delta(ScP s) { return s->deltaf; }
  static __device__ __forceinline__ float relax(ScP s) { return s->relaxf; }
  static __device__ __forceinline__ float relax_k(ScP s) { return s->relax_kf; }
  static __device__ __forceinline__ float amb_lo(ScP s, int r, int i) { return s->amb_lof[r][i]; }
  static __device__ __forceinline__ float amb_hi(ScP s, int r, int i) { return s->amb_hif[r][i]; }
  static __device__ __forceinline__ V3<float> acc_lo(const SMCRT_K Accel& A) { return {A.lof[0], A.lof[1], A.lof[2]}; }
  static __device__ __forceinline__ V3<float> acc_inv(const SMCRT_K Accel& A) { return {A.inv_cellf[0], A.inv_cellf[1], A.inv_cellf[2]}; }
  static __device__ __forceinline__ V3<float> acc_blo(const SMCRT_K Accel& A) { return {A.box_lof[0], A.box_lof[1], A.box_lof[2]}; }
  static __device__ __forceinline__ V3<float> acc_bhi(const SMCRT_K Accel& A) { return {A.box_hif[0], A.box_hif[1], A.box_hif[2]}; }
  static __device__ __forceinline__ float acc_margin(const SMCRT_K Accel& A) { return A.marginf; }
  static __device__ __forceinline__ float acc_cell_min(const SMCRT_K Accel& A) { return A.cell_minf; }
  static __device__ __forceinline__ float seg_err(ScP s) { return s->seg_errf; }
  // slack of a rate of approach: a few units in the last place
  static __device__ __forceinline__ float seg_eps() { return 0x1p-20f; }
};
template <>
struct Tab<double> {
  static __device__ __forceinline__ const SMCRT_K PrimD* prims(JobRef a) { return kptr(a.pd); }
  static __device__ __forceinline__ const SMCRT_K double* caps(JobRef a) { return kptr(a.acc_capd); }
  static __device__ __forceinline__ const SMCRT_K StepRec<double>* steps(JobRef a) { return kptr(a.step_d); }
  static __device__ __forceinline__ double hg_b(RegRef r) { return r.hg_b; }
  static __device__ __forceinline__ double hg_c(RegRef r) { return r.hg_c; }
  static __device__ __forceinline__ double hg_d(RegRef r) { return r.hg_d; }
  static __device__ __forceinline__ double k(RegRef r) { return r.k; }
  static __device__ __forceinline__ double inv_k(RegRef r) { return r.inv_k; }
  static __device__ __forceinline__ double mut(RegRef r) { return r.mut; }
  static __device__ __forceinline__ double inv_mut(RegRef r) { return r.inv_mut; }
  static __device__ __forceinline__ V3<double> bb_c(ScP s) { return {s->bb_c[0], s->bb_c[1], s->bb_c[2]}; }
  static __device__ __forceinline__ V3<double> bb_h(ScP s) { return {s->bb_h[0], s->bb_h[1], s->bb_h[2]}; }
  static __device__ __forceinline__ double bb_c(ScP s, int i) { return s->bb_c[i]; }
  static __device__ __forceinline__ double bb_h(ScP s, int i) { return s->bb_h[i]; }
  static __device__ __forceinline__ V3<double> g_lo(ScP s) { return {s->g_lo[0], s->g_lo[1], s->g_lo[2]}; }
  static __device__ __forceinline__ V3<double> g_inv(ScP s) { return {s->g_inv_d[0], s->g_inv_d[1], s->g_inv_d[2]}; }
  static __device__ __forceinline__ double g_d(ScP s, int i) { return s->g_d[i]; }
  static __device__ __forceinline__ double g_lo(ScP s, int i) { return s->g_lo[i]; }
  static __device__ __forceinline__ double g_hi(ScP s, int i) { return s->g_hi[i]; }
  static __device__ __forceinline__ double delta(ScP s) { return s->delta; }
  static __device__ __forceinline__ double relax(ScP s) { return s->relax; }
  static __device__ __forceinline__ double relax_k(ScP s) { return s->relax_k; }
  static __device__ __forceinline__ double amb_lo(ScP s, int r, int i) { return s->amb_lo[r][i]; }
  static __device__ __forceinline__ double amb_hi(ScP s, int r, int i) { return s->amb_hi[r][i]; }
  static __device__ __forceinline__ V3<double> acc_lo(const SMCRT_K Accel& A) { return {A.lo[0], A.lo[1], A.lo[2]}; }
  static __device__ __forceinline__ V3<double> acc_inv(const SMCRT_K Accel& A) { return {A.inv_cell[0], A.inv_cell[1], A.inv_cell[2]}; }
  static __device__ __forceinline__ V3<double> acc_blo(const SMCRT_K Accel& A) { return {A.box_lo[0], A.box_lo[1], A.box_lo[2]}; }
  static __device__ __forceinline__ V3<double> acc_bhi(const SMCRT_K Accel& A) { return {A.box_hi[0], A.box_hi[1], A.box_hi[2]}; }
  static __device__ __forceinline__ double acc_margin(const SMCRT_K Accel& A) { return A.margin; }
  static __device__ __forceinline__ double acc_cell_min(const SMCRT_K Accel& A) { return A.cell_min; }
  static __device__ __forceinline__ double seg_err(ScP s) { return s->seg_err; }
  static __device__ __forceinline__ double seg_eps() { return 1e-12; }
};

// exact Euclidean SDF of one primitive's shape in its own frame (Sec. 2.2;
// Eq. 3 for the sphere)
template <typename T, typename Params>
__device__ __forceinline__ T shape_of(int kind, const Params& v, V3<T> p) {
  const V3<T> q = p - mk(v[0], v[1], v[2]);
  if (kind == kSphere) return tsqrt(fdot(q, q)) - v[3];
  if (kind == kBox) {
    const T ex = tabs(q.x) - v[3], ey = tabs(q.y) - v[4], ez = tabs(q.z) - v[5];
    const V3<T> o = mk(tmax(ex, T(0)), tmax(ey, T(0)), tmax(ez, T(0)));
    return tsqrt(fdot(o, o)) + tmin(tmax(ex, tmax(ey, ez)), T(0));
  }
  const V3<T> e = mk(v[3], v[4], v[5]);
  if (kind == kTorus) {  // e unit axis, v[6] = ring radius R, v[7] = tube radius r
    const T x = fdot(q, e);
    const V3<T> rad = fback(q, x, e);
    const T rho = tsqrt(fdot(rad, rad)) - v[6];
    return tsqrt(tfma(x, x, rho * rho)) - v[7];
  }
  if (kind == kCapsule) {  // e = b - a, v[6] = 1/|b-a|^2
    const T t = tclamp(fdot(q, e) * v[6], T(0), T(1));
    const V3<T> d = fback(q, t, e);
    return tsqrt(fdot(d, d)) - v[7];
  }
  // capped cylinder: e unit axis, v[6] = L, v[7] = L/2, v[8] = r
  const T x = fdot(q, e);
  const V3<T> rad = fback(q, x, e);
  const T q1 = tsqrt(fdot(rad, rad)) - v[8];
  const T q2 = tabs(x - v[7]) - v[7];
  const T o1 = tmax(q1, T(0)), o2 = tmax(q2, T(0));
  return tmin(tmax(q1, q2), T(0)) + tsqrt(sum_sq(o1, o2));
}
template <typename T>
__device__ __forceinline__ T shape_sdf(const SMCRT_K Prim<T>* P, int i, V3<T> p) {
  const SMCRT_K T* v = P[i].v;
  return shape_of<T>(P[i].kind, v, p);
}

// sin and cos of a twist or displacement angle (moderate arguments):
// Cody-Waite reduction by pi/2, split into the precision's nearest value and
// its residual, to r in [-pi/4, pi/4], then the Taylor series of sin and cos
// to r^17 / r^16 (FP64: last term < 4e-18) or r^11 / r^10 (FP32: < 1e-9),
// evaluated by Horner's rule; the quadrant n mod 4 picks signs and order.
// Kept in registers: the library routine's reduction for huge arguments
// needs a stack array, which in the sphere-tracing loop moved other
// values to scratch.
template <typename T>
__device__ __forceinline__ void tsincos(T a, T* sn, T* cs) {
  const T n = rint(a * T(0.63661977236758134308));  // 2/pi
  // pi/2 = hi + lo: FP64 0x3FF921FB54442D18 + 6.1232e-17, FP32 0x3FC90FDB - 4.3711e-8
  const T hi = sizeof(T) == 8 ? T(1.5707963267948966) : T(1.57079637050628662109375);
  const T lo = sizeof(T) == 8 ? T(6.123233995736766e-17) : T(-4.371139000186241e-08);
  const T r = (a - n * hi) - n * lo;
  const T r2 = r * r;
  T s, c;
  if constexpr (sizeof(T) == 8) {
    s = T(1) / T(355687428096000);
    s = s * -r2 + T(1) / T(1307674368000);
    s = s * -r2 + T(1) / T(6227020800);
    s = s * -r2 + T(1) / T(39916800);
    s = s * -r2 + T(1) / T(362880);
    s = s * -r2 + T(1) / T(5040);
    s = s * -r2 + T(1) / T(120);
    s = s * -r2 + T(1) / T(6);
    s = r - r * r2 * s;
    c = T(1) / T(20922789888000);
    c = c * -r2 + T(1) / T(87178291200);
    c = c * -r2 + T(1) / T(479001600);
    c = c * -r2 + T(1) / T(3628800);
    c = c * -r2 + T(1) / T(40320);
    c = c * -r2 + T(1) / T(720);
    c = c * -r2 + T(1) / T(24);
    c = c * -r2 + T(1) / T(2);
    c = T(1) - r2 * c;
  } else {
    s = T(1) / T(39916800);
    s = s * -r2 + T(1) / T(362880);
    s = s * -r2 + T(1) / T(5040);
    s = s * -r2 + T(1) / T(120);
    s = s * -r2 + T(1) / T(6);
    s = r - r * r2 * s;
    c = T(1) / T(3628800);
    c = c * -r2 + T(1) / T(40320);
    c = c * -r2 + T(1) / T(720);
    c = c * -r2 + T(1) / T(24);
    c = c * -r2 + T(1) / T(2);
    c = T(1) - r2 * c;
  }
  const int q = ((int)n) & 3;
  *sn = q == 0 ? s : (q == 1 ? c : (q == 2 ? -s : -c));
  *cs = q == 0 ? c : (q == 1 ? -s : (q == 2 ? -c : s));
}

// SDF of primitive i (Sec. 2.2: SDFs are translated, rotated, scaled,
// twisted and bent).  Placement with uniform scale keeps the distance exact
// (times s), and so do rounding and the onion shell.  A twist or a bend
// keeps the sign; inside its bounding cylinder (radius rho) the distance is
// divided by the untwist (unbend) map's Lipschitz bound there, the largest
// singular value of its Jacobian, (k rho + sqrt((k rho)^2 + 4)) / 2 for a
// twist and 1 + k rho for a bend; outside it the distance to the cylinder
// is used.  The flags are the
// same for every lane (primitives are visited in a wave-uniform order).
// distance from (x, y) to the segment (ax, ay)-(bx, by)
template <typename T>
__device__ __forceinline__ T seg2_dist(T x, T y, T ax, T ay, T bx, T by) {
  const T dx = bx - ax, dy = by - ay, px = x - ax, py = y - ay;
  const T t = tclamp((px * dx + py * dy) / (dx * dx + dy * dy), T(0), T(1));
  const T ex = px - t * dx, ey = py - t * dy;
  return tsqrt(ex * ex + ey * ey);
}

// distance from p to the segment a-b
template <typename T>
__device__ __forceinline__ T seg3_dist(V3<T> p, V3<T> a, V3<T> b) {
  const V3<T> ba = b - a, pa = p - a;
  const T t = tclamp(dot(pa, ba) / dot(ba, ba), T(0), T(1));
  const V3<T> d = pa - t * ba;
  return tsqrt(dot(d, d));
}

// further gallery shapes in their own frame (Sec. 2.2, Fig. 1's basic
// shapes): capped cone, octahedron and hexagonal prism (exact distances),
// ellipsoid (a lower bound with the exact sign)
template <typename T>
__device__ __forceinline__ T further_shape_sdf(const SMCRT_K Prim<T>* P, int i, V3<T> p) {
  const int kind = P[i].kind;
  const SMCRT_K T* v = P[i].v;
  const V3<T> q = p - mk(v[0], v[1], v[2]);
  if (kind == kCone) {  // (axial x, radial y) half plane: the two caps and the slanted side
    const V3<T> e = mk(v[3], v[4], v[5]);
    const T L = v[6], ra = v[7], rb = v[8];
    const T x = fdot(q, e);
    const V3<T> rad = q - x * e;
    const T y = tsqrt(fdot(rad, rad));
    const T d = tmin(tmin(seg2_dist(x, y, T(0), T(0), T(0), ra), seg2_dist(x, y, L, T(0), L, rb)),
                     seg2_dist(x, y, T(0), ra, L, rb));
    const bool inside = x > T(0) && x < L && y < ra + (rb - ra) * x / L;
    return inside ? -d : d;
  }
  if (kind == kOctahedron) {  // by symmetry the face in the positive octant
    const T s = v[3];
    const V3<T> a = mk(tabs(q.x), tabs(q.y), tabs(q.z));
    const T m = a.x + a.y + a.z - s;
    const T third = m * T(1.0 / 3.0);
    if (m <= T(0) || (a.x >= third && a.y >= third && a.z >= third)) return m * T(0.57735026918962576451);
    const V3<T> v0 = mk(s, T(0), T(0)), v1 = mk(T(0), s, T(0)), v2 = mk(T(0), T(0), s);
    return tmin(tmin(seg3_dist(a, v0, v1), seg3_dist(a, v1, v2)), seg3_dist(a, v2, v0));
  }
  if (kind == kHexPrism) {  // first quadrant: edges (R,0)-(R/2,h) and (R/2,h)-(-R/2,h)
    const T h = v[3], hz = v[4], R = v[5];
    const T x = tabs(q.x), y = tabs(q.y);
    T d2 = tmin(seg2_dist(x, y, R, T(0), T(0.5) * R, h), seg2_dist(x, y, T(0.5) * R, h, T(-0.5) * R, h));
    if (y < h && T(1.7320508075688772935) * x + y < T(2) * h) d2 = -d2;
    const T dz = tabs(q.z) - hz;
    const T o1 = tmax(d2, T(0)), o2 = tmax(dz, T(0));
    return tmin(tmax(d2, dz), T(0)) + tsqrt(tfma(o2, o2, o1 * o1));
  }
  // ellipsoid: rmin (|q / r| - 1), 1-Lipschitz and zero on the surface
  const V3<T> u = mk(q.x * v[3], q.y * v[4], q.z * v[5]);
  return v[6] * (tsqrt(fdot(u, u)) - T(1));
}

// SDF of a placed or modified primitive.  Inlined into the walk's steps and
// called from elsewhere, it should round the same: the sums of products here
// and in the basic shapes are explicit fma.  Those of the further shapes and of
// tsincos are left to the compiler, which fuses them alike in both (written
// out, shared products round otherwise than they have, and the FP64 kernel
// spills 45 registers instead of 27).
template <typename T>
__device__ __forceinline__ T placed_prim(const SMCRT_K Prim<T>* P, int i, V3<T> p) {
  hold(p.x);
  hold(p.y);
  hold(p.z);
  const SMCRT_K Prim<T>& Q = P[i];
  const int fl = Q.flags;
  V3<T> q = p;
  if (fl & kPlaced) {
    const V3<T> d = p - mk(Q.t[0], Q.t[1], Q.t[2]);
    q = mk(fdot(mk(Q.m[0], Q.m[1], Q.m[2]), d), fdot(mk(Q.m[3], Q.m[4], Q.m[5]), d), fdot(mk(Q.m[6], Q.m[7], Q.m[8]), d));
  }
  // repetition: to the nearest copy; b = distance to the nearest face of its
  // cell with another copy behind it
  T b = tinf<T>();
  if (fl & kRepeated) {
    T c3[3] = {q.x, q.y, q.z};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int n = Q.rep_n[a];
      const T c = Q.rep_c[a], half = T(0.5) * T(n - 1) * c;
      // clamp before converting: a far point must not overflow the int
      const int k = (int)tclamp(floor(tfma(c, T(0.5) * T(n - 1), c3[a]) / c + T(0.5)), T(0), T(n - 1));
      c3[a] -= tfma(T(k), c, -half);
      if (c3[a] > T(0) && k < n - 1) b = tmin(b, T(0.5) * c - c3[a]);
      if (c3[a] < T(0) && k > 0) b = tmin(b, T(0.5) * c + c3[a]);
    }
    q = mk(c3[0], c3[1], c3[2]);
  }
  T dcyl = T(0);
  if (fl & kTwisted) {  // distance to the bounding cylinder, then untwist by -k z (unbend: -k x) about z
    const T q1 = tsqrt(tfma(q.x, q.x, q.y * q.y)) - Q.twist_rho;
    const T q2 = tabs(q.z - Q.twist_zc) - Q.twist_zh;
    const T o1 = tmax(q1, T(0)), o2 = tmax(q2, T(0));
    dcyl = tmin(tmax(q1, q2), T(0)) + tsqrt(tfma(o1, o1, o2 * o2));
    T sn, cs;
    tsincos(-Q.twist_k * ((fl & kBent) ? q.x : q.z), &sn, &cs);
    q = mk(tfma(cs, q.x, -(sn * q.y)), tfma(sn, q.x, cs * q.y), q.z);
  }
  const V3<T> e = mk(q.x - tclamp(q.x, -Q.elong[0], Q.elong[0]), q.y - tclamp(q.y, -Q.elong[1], Q.elong[1]),
                     q.z - tclamp(q.z, -Q.elong[2], Q.elong[2]));
  T d = ((fl & kFurtherShape) ? further_shape_sdf(P, i, e) : shape_sdf(P, i, e)) - Q.round_r;
  if (Q.onion_t > T(0)) d = tabs(d) - Q.onion_t;
  if (Q.disp_a > T(0)) {
    T sx, cx, sy, cy, sz, cz;
    tsincos(Q.disp_f * q.x, &sx, &cx);
    tsincos(Q.disp_f * q.y, &sy, &cy);
    tsincos(Q.disp_f * q.z, &sz, &cz);
    d = tfma(Q.disp_a * sx * sy, sz, d) * Q.disp_inv_lip;
  }
  if (fl & kTwisted) d = dcyl > T(0) ? dcyl : d * Q.inv_lip;
  if (fl & kRepeated) d = tmin(d, Q.rep_gap + b);
  if (fl & kPlaced) d *= Q.s;
  hold(d);
  return d;
}
// The same as a function, for the rarer places.  UNI: i is the same for every
// lane.  A function's arguments arrive in vector registers; taken back to
// scalar ones, the parameters are scalar loads instead of vector loads that
// wait for the wave's atomics: 2e5 packets of the gallery scene 23 % less
// time, with the steps' evaluations inlined 6 % less again, inlined everywhere
// 3 % more.
template <typename T, bool UNI>
__device__ __attribute__((noinline)) T placed_prim_sdf(const SMCRT_K Prim<T>* P, int i, V3<T> p) {
  if constexpr (UNI) {
    const uint64_t v = (uint64_t)P;
    P = (const SMCRT_K Prim<T>*)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32)) << 32) |
                                 (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v));
    i = __builtin_amdgcn_readfirstlane(i);
  }
  return placed_prim<T>(P, i, p);
}

// XF: the scene has placed or modified primitives.  Scenes without them
// run kernels that never call placed_prim_sdf: a call in the sphere-tracing
// loop makes the caller keep its live values out of the registers the
// callee may use, which pushed the FP32 walk over its register budget.
template <typename T, bool XF, bool UNI = true>
__device__ __forceinline__ T prim_sdf(const SMCRT_K Prim<T>* P, int i, V3<T> p) {
  if constexpr (XF) {
    if (P[i].flags != 0) return placed_prim_sdf<T, UNI>(P, i, p);
  }
  return shape_sdf(P, i, p);
}

// polynomial smooth union of two distances, its roundings fixed like fdot's
template <typename T>
__device__ __forceinline__ T smooth_min(T d, T b, T k, T inv_k) {
  const T h = tclamp(tfma(T(0.5) * (b - d), inv_k, T(0.5)), T(0), T(1));
  const T g = T(1) - h;
  return tfma(-(k * h), g, tfma(h, d, g * b));
}

// region SDF from its primitives in order (CSG of Sec. 2.2): union (min),
// polynomial smooth union, intersection (max) or difference, the first
// primitive minus the others (max(d, -d_i)).  Intersection and difference
// are lower bounds of the distance with Lipschitz constant 1, so sphere
// tracing stays conservative.
template <typename T, bool XF>
__device__ __forceinline__ T region_sdf(JobRef a, RegRef R, V3<T> p) {
  const SMCRT_K Prim<T>* P = Tab<T>::prims(a);
  const int op = R.op;  // wave uniform: one loop, primitive SDFs inlined once
  T d = prim_sdf<T, XF>(P, R.first, p);
  for (int i = 1; i < R.count; ++i) {
    const T b = prim_sdf<T, XF>(P, R.first + i, p);
    if (op == kSmoothUnion) {
      d = smooth_min(d, b, Tab<T>::k(R), Tab<T>::inv_k(R));
    } else {
      const T nb = op == kSubtract ? -b : b;
      d = op == kUnion ? tmin(d, nb) : tmax(d, nb);
    }
  }
  return d;
}

// capsule SDF from a compact record c = (a, b - a, 1/|b - a|^2, r): the
// capsule branch of shape_of, operation for operation
template <typename T>
__device__ __forceinline__ T cap_sdf(T a0, T a1, T a2, T e0, T e1, T e2, T inv, T r, V3<T> p) {
  const V3<T> q = p - mk(a0, a1, a2);
  const V3<T> e = mk(e0, e1, e2);
  const T t = tclamp(fdot(q, e) * inv, T(0), T(1));
  const V3<T> d = fback(q, t, e);
  return tsqrt(fdot(d, d)) - r;
}

// An evaluation record in scalar registers.
typedef uint32_t U16 __attribute__((ext_vector_type(16)));
template <typename T>
struct StepV;
template <>
struct StepV<float> {
  U16 w;
  __device__ __forceinline__ int bits() const { return (int)w[0]; }
  __device__ __forceinline__ int index() const { return (int)w[1]; }
  __device__ __forceinline__ uint32_t word(int i) const { return w[i & 15]; }
  __device__ __forceinline__ float operator[](int k) const { return __builtin_bit_cast(float, (uint32_t)w[2 + k]); }
  __device__ __forceinline__ float k() const { return (*this)[10]; }
  __device__ __forceinline__ float inv_k() const { return (*this)[11]; }
};
template <>
struct StepV<double> {
  U16 w, x;
  __device__ __forceinline__ int bits() const { return (int)w[0]; }
  __device__ __forceinline__ int index() const { return (int)w[1]; }
  __device__ __forceinline__ uint32_t word(int i) const { return i < 16 ? w[i & 15] : x[i & 15]; }
  __device__ __forceinline__ double operator[](int k) const {
    return __builtin_bit_cast(double, (uint64_t)word(2 + 2 * k) | ((uint64_t)word(3 + 2 * k) << 32));
  }
  __device__ __forceinline__ double k() const { return (*this)[10]; }
  __device__ __forceinline__ double inv_k() const { return (*this)[11]; }
};
__device__ __forceinline__ StepV<float> load_step(const SMCRT_K StepRec<float>* r) {
  return {*reinterpret_cast<const SMCRT_K U16*>(r)};
}
__device__ __forceinline__ StepV<double> load_step(const SMCRT_K StepRec<double>* r) {
  const SMCRT_K U16* q = reinterpret_cast<const SMCRT_K U16*>(r);
  return {q[0], q[1]};
}

// What a query of the acceleration grid needs, from the scene header or from
// the region's evaluation record.
template <typename T>
struct GridV {
  V3<T> lo, ic;
  T margin, cell_min;
  int dx, dy, dz;
  uint32_t first, n;
  uint64_t capacity;
  bool caps;
};
template <typename T>
__device__ __forceinline__ GridV<T> grid_of(const SMCRT_K Accel& A) {
  return {Tab<T>::acc_lo(A), Tab<T>::acc_inv(A), Tab<T>::acc_margin(A), Tab<T>::acc_cell_min(A), A.dims[0], A.dims[1],
          A.dims[2], (uint32_t)A.first_prim, (uint32_t)A.n_prims, A.capacity, A.caps != 0};
}
template <typename T>
__device__ __forceinline__ GridV<T> grid_of(const StepV<T>& r) {  // AccelRec
  constexpr int w = 2 + 8 * (int)sizeof(T) / 4;
  return {mk(r[0], r[1], r[2]), mk(r[3], r[4], r[5]), r[6], r[7], (int)r.word(w), (int)r.word(w + 1), (int)r.word(w + 2),
          (uint32_t)r.index(), r.word(w + 3), (uint64_t)r.word(w + 4) | ((uint64_t)r.word(w + 5) << 32),
          (r.bits() & kStepCaps) != 0};
}

// Lower bound of the accelerated region's SDF at p in a cell that lists no
// primitive, from the cell's ring distance k (in cells) to the nearest cell
// that lists one: every surface point lies in such a cell, so the surface is
// at least k - 1 whole cells plus p's way to its own cell's faces away (the
// smallest side counted; cell coordinates cx, cy, cz of p and its cell
// ix, iy, iz).  Never below the margin; a relative 2^-20 less against
// rounding.
template <typename T>
__device__ __forceinline__ T ring_bound(JobRef a, T margin, T cell_min, int c, T cx, T cy, T cz, int ix, int iy, int iz) {
  if (a.acc_rings == nullptr) return margin;
  const uint32_t k = kptr(a.acc_rings)[c];
  const T fx = cx - T(ix), fy = cy - T(iy), fz = cz - T(iz);
  const T f = tmin(tmin(tmin(fx, T(1) - fx), tmin(fy, T(1) - fy)), tmin(fz, T(1) - fz));
  const T r = (T(k) - T(1) + tmax(f, T(0))) * cell_min * (T(1) - T(0x1p-20));
  return tmax(margin, r);
}

// Where p lies in the grid of the accelerated region.  True when its cell
// lists primitives: ids[*b, *e).  Else *d is the region's distance bound
// there: outside the grid box (which is the primitives' box grown by the
// margin) the distance to the primitives' box, in an empty cell its ring's.
template <typename T>
__device__ __forceinline__ bool grid_cell(JobRef a, const GridV<T>& G, V3<T> p, uint32_t* b, uint32_t* e, T* d) {
  const T cx = (p.x - G.lo.x) * G.ic.x, cy = (p.y - G.lo.y) * G.ic.y, cz = (p.z - G.lo.z) * G.ic.z;
  const int dx = G.dx, dy = G.dy, dz = G.dz;
  if (!(cx >= T(0) && cy >= T(0) && cz >= T(0) && cx < T(dx) && cy < T(dy) && cz < T(dz))) {
    const SMCRT_K Accel& A = kptr(a.sc)->acc;
    const V3<T> bl = Tab<T>::acc_blo(A), bh = Tab<T>::acc_bhi(A);
    const V3<T> o = mk(tmax(tmax(bl.x - p.x, p.x - bh.x), T(0)), tmax(tmax(bl.y - p.y, p.y - bh.y), T(0)),
                       tmax(tmax(bl.z - p.z, p.z - bh.z), T(0)));
    *d = tsqrt(dot(o, o));
    return false;
  }
  int ix = (int)cx, iy = (int)cy, iz = (int)cz;
  ix = ix < dx ? ix : dx - 1;
  iy = iy < dy ? iy : dy - 1;
  iz = iz < dz ? iz : dz - 1;
  const int c = ix + dx * (iy + dy * iz);
  const SMCRT_K uint32_t* offs = kptr(a.acc_offsets);
  const uint32_t first = offs[c], last = offs[c + 1];
  *b = first;
  *e = (uint64_t)last < G.capacity ? last : (uint32_t)G.capacity;
  if (*b < *e) return true;
  *d = ring_bound<T>(a, G.margin, G.cell_min, c, cx, cy, cz, ix, iy, iz);
  return false;
}

// SDF of the accelerated region through its uniform grid: min(margin, min
// over the primitives listed in p's cell).  Equal to the region SDF where
// that is below the margin, a lower bound elsewhere; outside the grid box
// (which is the primitives' box grown by the margin) the distance to the
// primitives' box is the lower bound.  Every index is checked.  Regions of
// plain capsules read their compact records: from the workgroup's LDS
// table when lds is given (FP32 staged walk), else from global memory.
template <typename T, bool XF>
__device__ __forceinline__ T accel_sdf(JobRef a, const GridV<T>& G, V3<T> p, LdsCaps lds = nullptr) {
  uint32_t b, e;
  T d;
  if (!grid_cell<T>(a, G, p, &b, &e, &d)) return d;
  const SMCRT_K uint32_t* ids = kptr(a.acc_ids);
  d = G.margin;
  if (G.caps) {
    if constexpr (sizeof(T) == 4) {
      if (lds) {
        for (uint32_t i = b; i < e; ++i) {
          const uint32_t id = ids[i] - G.first, k = id < G.n ? id : 0u;
          const F4 x = lds[2 * k], y = lds[2 * k + 1];
          const T v = cap_sdf<T>(x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w, p);
          d = id < G.n ? tmin(d, v) : d;
        }
        return d;
      }
    }
    const SMCRT_K T* C = Tab<T>::caps(a);
    for (uint32_t i = b; i < e; ++i) {
      const uint32_t id = ids[i] - G.first, k = id < G.n ? id : 0u;
      const SMCRT_K T* c = C + 8 * (size_t)k;
      const T v = cap_sdf<T>(c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7], p);
      d = id < G.n ? tmin(d, v) : d;
    }
    return d;
  }
  const SMCRT_K Prim<T>* P = Tab<T>::prims(a);
  for (uint32_t i = b; i < e; ++i) {
    const uint32_t id = ids[i];
    if (id - G.first < G.n) d = tmin(d, prim_sdf<T, XF, false>(P, (int)id, p));
  }
  return d;
}

// SDF of region r (through the grid when r is the accelerated region)
template <typename T, bool XF>
__device__ __forceinline__ T region_dist(JobRef a, int r, V3<T> p, LdsCaps lds = nullptr) {
  if (r == a.acc_region) return accel_sdf<T, XF>(a, grid_of<T>(kptr(a.sc)->acc), p, lds);
  return region_sdf<T, XF>(a, kptr(a.sc)->reg[r], p);
}

// Distance of p to the nearest surface: the smallest |region_dist| over the
// regions, by the scene's evaluation records.  A lone wave waits for every
// scalar load it needs; walked through the region, then its primitive's kind,
// then its parameters, that is four or five waits in a row per region.  A
// record holds all of it in whole cache lines, and the next one is on its way
// while this one is worked on.  (With the packets' region rows in LDS: 1e5
// packets of the 50^3 sphere 8 % less time.)
template <typename T, bool XF>
__device__ __forceinline__ T walk_distance(JobRef a, const SMCRT_K StepRec<T>* rec, int n_steps, V3<T> p,
                                           LdsCaps lds) {
  StepV<T> cur = load_step(rec);
  T dmin = tinf<T>(), d = T(0);
  for (int i = 1;; ++i) {
    const bool more = i < n_steps;
    const StepV<T> next = load_step(rec + (more ? i : 0));
    const int bits = cur.bits(), kind = bits & kStepKind, op = bits >> kStepOp;
    if (kind == kStepAccel) {
      d = accel_sdf<T, XF>(a, grid_of<T>(cur), p, lds);
    } else {
      T b;
      if (XF && (bits & kStepPlaced)) b = placed_prim<T>(Tab<T>::prims(a), cur.index(), p);
      else b = shape_of<T>(kind, cur, p);
      if (bits & kStepFirst) {
        d = b;
      } else if (op == kSmoothUnion) {
        d = smooth_min(d, b, cur.k(), cur.inv_k());
      } else {
        const T nb = op == kSubtract ? -b : b;
        d = op == kUnion ? tmin(d, nb) : tmax(d, nb);
      }
    }
    if (bits & kStepLast) dmin = tmin(dmin, tabs(d));
    if (!more) return dmin;
    cur = next;
  }
}

// owner of a point: the highest-index region with a negative SDF, else the
// ambient slot n_regions
template <typename T, bool XF>
__device__ __forceinline__ int region_of(JobRef a, V3<T> p) {
  ScP sc = kptr(a.sc);
  const int nr = sc->n_regions;
  int owner = nr;
  for (int r = nr - 1; r >= 0; --r) {
    if (region_dist<T, XF>(a, r, p) < T(0)) {
      owner = r;
      break;
    }
  }
  return owner;
}

// Outside the simulation volume (Sec. 2.3: escape when the volume's box
// SDF is positive).  The box SDF is positive exactly when the largest of
// |q_i| - h_i is, so the sign needs no square root; volume_face: 2*axis +
// side of that largest component, the face the packet left through.
template <typename T>
__device__ __forceinline__ bool outside_volume(ScP sc, V3<T> p) {
  const V3<T> c = Tab<T>::bb_c(sc), h = Tab<T>::bb_h(sc);
  const V3<T> q = p - c;
  return tmax(tabs(q.x) - h.x, tmax(tabs(q.y) - h.y, tabs(q.z) - h.z)) > T(0);
}
template <typename T>
__device__ __forceinline__ int volume_face(ScP sc, V3<T> p) {
  const V3<T> c = Tab<T>::bb_c(sc), h = Tab<T>::bb_h(sc);
  const V3<T> q = p - c;
  const T ex = tabs(q.x) - h.x, ey = tabs(q.y) - h.y, ez = tabs(q.z) - h.z;
  int ax = 0;
  T best = ex;
  if (ey > best) { best = ey; ax = 1; }
  if (ez > best) { best = ez; ax = 2; }
  const T qa = ax == 0 ? q.x : (ax == 1 ? q.y : q.z);
  return 2 * ax + (qa > T(0) ? 1 : 0);
}

// Ambient skip: outside every region, the straight path from p along u
// cuts no surface before it enters the box of some region's surface; when
// it enters none inside the volume, only the volume's boundary lies ahead.
// Returns the path to the first such box, or delta past the boundary; 0
// when p is inside a box.  (u == 0 on an axis: the box is met only when p
// lies between its planes.)
template <typename T>
__device__ __forceinline__ T ambient_free(ScP sc, int nr, V3<T> p, V3<T> u, T delta) {
  // (the compiler would take the divisions out of the loop of steps, few of
  // which come this way)
  hold(u.x);
  hold(u.y);
  hold(u.z);
  const V3<T> c = Tab<T>::bb_c(sc), h = Tab<T>::bb_h(sc);
  const T pv[3] = {p.x, p.y, p.z}, uv[3] = {u.x, u.y, u.z};
  const T cv[3] = {c.x, c.y, c.z}, hv[3] = {h.x, h.y, h.z};
  T rv[3];
  T t = tinf<T>();
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    rv[i] = T(1) / uv[i];
    if (uv[i] != T(0)) t = tmin(t, ((uv[i] > T(0) ? cv[i] + hv[i] : cv[i] - hv[i]) - pv[i]) * rv[i]);
  }
  t += delta;
  for (int r = 0; r < nr; ++r) {
    T t0 = T(0), t1 = t;
    bool hit = true;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const T lo = Tab<T>::amb_lo(sc, r, i), hi = Tab<T>::amb_hi(sc, r, i);
      if (uv[i] == T(0)) {
        hit = hit && pv[i] >= lo && pv[i] <= hi;
      } else {
        const T ta = (lo - pv[i]) * rv[i], tb = (hi - pv[i]) * rv[i];
        t0 = tmax(t0, tmin(ta, tb));
        t1 = tmin(t1, tmax(ta, tb));
      }
    }
    if (hit && t0 <= t1) t = t0;
  }
  return t;
}

// ---- segment tracing (Sec. 5 names it beside enhanced sphere tracing as a
// cure for the many small steps of rays that run along surfaces).  Outside
// a convex shape the exact distance along a ray, f(t) = d(p + t u), is a
// convex function of t and never falls below its tangent f(0) - c t, where
// c = -grad d . u is the rate at which the ray approaches the shape: the ray
// cannot reach the shape before f(0) / c, nor ever when c <= 0.  A union is
// reached when one member is (the smallest bound), an intersection only when
// every member is (the largest bound), a subtraction not before its first
// member.  Rounding: f(0) is taken less err, the scene's bound on the
// rounding of a distance, and c more err / f(0) (the gradient is the
// direction of a difference known to err) plus a few units in the last
// place.

// the length a ray runs before it can reach a convex shape at distance a
// that it approaches at rate c = -dv / l (dv = v . u for a vector v of
// length l > 0 from the nearest surface point towards p), with the rounding
// slack: (a - err) / (c + err / a + eps), taken as l a (a - err) / (l (err
// + eps a) - a dv), one division.  0 when a is within the rounding (or the
// rate is not a number), infinite when the ray moves away.
template <typename T>
__device__ __forceinline__ T tangent_bound(T a, T dv, T l, T err) {
  if (!(a > err)) return T(0);
  const T den = l * (err + Tab<T>::seg_eps() * a) - a * dv;
  if (den > T(0)) return tdiv(l * a * (a - err), den);
  return den <= T(0) ? tinf<T>() : T(0);
}

// distance of a plain convex primitive (sphere, box, capsule or capped
// cylinder, unplaced and unmodified) at p, by the operations of shape_of, and the ray's rate of approach to it as -(*dv) / (*l): v points from
// the nearest surface point towards p (meaningful outside the shape)
template <typename T>
__device__ __forceinline__ T convex_sdf_rate(const SMCRT_K Prim<T>* P, int i, V3<T> p, V3<T> u, T* dv, T* l) {
  const int kind = P[i].kind;
  const SMCRT_K T* v = P[i].v;
  const V3<T> q = p - mk(v[0], v[1], v[2]);
  if (kind == kSphere) {
    *l = tsqrt(fdot(q, q));
    *dv = dot(q, u);
    return *l - v[3];
  }
  if (kind == kBox) {
    const T ex = tabs(q.x) - v[3], ey = tabs(q.y) - v[4], ez = tabs(q.z) - v[5];
    const V3<T> o = mk(tmax(ex, T(0)), tmax(ey, T(0)), tmax(ez, T(0)));
    *l = tsqrt(fdot(o, o));
    *dv = (q.x < T(0) ? -o.x : o.x) * u.x + (q.y < T(0) ? -o.y : o.y) * u.y + (q.z < T(0) ? -o.z : o.z) * u.z;
    return *l + tmin(tmax(ex, tmax(ey, ez)), T(0));
  }
  const V3<T> e = mk(v[3], v[4], v[5]);
  if (kind == kCapsule) {
    const T t = tclamp(fdot(q, e) * v[6], T(0), T(1));
    const V3<T> d = fback(q, t, e);
    *l = tsqrt(fdot(d, d));
    *dv = dot(d, u);
    return *l - v[7];
  }
  // capped cylinder, in the half plane of (radial, axial) coordinates: v =
  // o1 rad / rho +/- o2 e, scaled by rho when o1 > 0
  const T x = fdot(q, e);
  const V3<T> rad = fback(q, x, e);
  const T rho = tsqrt(fdot(rad, rad));
  const T q1 = rho - v[8];
  const T q2 = tabs(x - v[7]) - v[7];
  const T o1 = tmax(q1, T(0)), o2 = tmax(q2, T(0));
  const T len = tsqrt(sum_sq(o1, o2));
  const T sc = o1 > T(0) ? rho : T(1);
  *l = sc * len;
  *dv = o1 * dot(rad, u) + (x > v[7] ? o2 : -o2) * sc * dot(e, u);
  return tmin(tmax(q1, q2), T(0)) + len;
}

// the accelerated region's distance (accel_sdf's value) and in *tb the
// way along u to its surface: inside the grid, the capsules listed in p's
// cell bound it by their tangents, and every other primitive lies farther
// than the margin; outside the grid (and for regions without a rule) the
// distance alone
template <typename T, bool XF>
__device__ __forceinline__ T accel_seg(JobRef a, V3<T> p, V3<T> u, T err, T* tb) {
  const SMCRT_K Accel& A = kptr(a.sc)->acc;
  const int rule = kptr(a.sc)->reg[A.region].seg;
  const V3<T> lo = Tab<T>::acc_lo(A), ic = Tab<T>::acc_inv(A);
  const T cx = (p.x - lo.x) * ic.x, cy = (p.y - lo.y) * ic.y, cz = (p.z - lo.z) * ic.z;
  const int dx = A.dims[0], dy = A.dims[1], dz = A.dims[2];
  if (rule != kSegUnion || !(cx >= T(0) && cy >= T(0) && cz >= T(0) && cx < T(dx) && cy < T(dy) && cz < T(dz))) {
    const T d = accel_sdf<T, XF>(a, grid_of<T>(A), p);
    *tb = tabs(d);
    return d;
  }
  int ix = (int)cx, iy = (int)cy, iz = (int)cz;
  ix = ix < dx ? ix : dx - 1;
  iy = iy < dy ? iy : dy - 1;
  iz = iz < dz ? iz : dz - 1;
  const int cell = ix + dx * (iy + dy * iz);
  const SMCRT_K uint32_t* offs = kptr(a.acc_offsets);
  const SMCRT_K uint32_t* ids = kptr(a.acc_ids);
  const uint32_t b = offs[cell];
  uint64_t e = offs[cell + 1];
  e = e < A.capacity ? e : A.capacity;
  if (b >= e) {
    const T d = ring_bound<T>(a, Tab<T>::acc_margin(A), Tab<T>::acc_cell_min(A), cell, cx, cy, cz, ix, iy, iz);
    *tb = d;
    return d;
  }
  const uint32_t lo_id = (uint32_t)A.first_prim, hi_id = (uint32_t)(A.first_prim + A.n_prims);
  T d = Tab<T>::acc_margin(A), t = d;
  if (A.caps) {
    const SMCRT_K T* C = Tab<T>::caps(a);
    for (uint64_t i = b; i < e; ++i) {
      const uint32_t id = ids[i];
      if (id >= lo_id && id < hi_id) {
        const SMCRT_K T* r = C + 8 * (size_t)(id - lo_id);
        const V3<T> q = p - mk(r[0], r[1], r[2]);
        const V3<T> ax = mk(r[3], r[4], r[5]);
        const T s = tclamp(fdot(q, ax) * r[6], T(0), T(1));
        const V3<T> w = fback(q, s, ax);
        const T l = tsqrt(fdot(w, w));
        const T di = l - r[7];
        d = tmin(d, di);
        t = tmin(t, tangent_bound<T>(di, dot(w, u), l, err));
      }
    }
  } else {
    const SMCRT_K Prim<T>* P = Tab<T>::prims(a);
    for (uint64_t i = b; i < e; ++i) {
      const uint32_t id = ids[i];
      if (id >= lo_id && id < hi_id) {
        T dv, l;
        const T di = convex_sdf_rate<T>(P, (int)id, p, u, &dv, &l);
        d = tmin(d, di);
        t = tmin(t, tangent_bound<T>(di, dv, l, err));
      }
    }
  }
  *tb = d > T(0) ? tmax(d, t) : tabs(d);
  return d;
}

// distance of region r at p (region_dist's value) and in *tb a length the
// ray along u runs before it can meet the region's surface: from outside a
// region with a rule, the tangent bounds of its members; else the
// distance's magnitude
template <typename T, bool XF>
__device__ __forceinline__ T region_seg(JobRef a, int r, V3<T> p, V3<T> u, T err, T* tb) {
  if (r == a.acc_region) return accel_seg<T, XF>(a, p, u, err, tb);
  const SMCRT_K Region& R = kptr(a.sc)->reg[r];
  const int rule = R.seg;  // wave uniform
  if (rule == kSegNone) {
    const T d = region_sdf<T, XF>(a, R, p);
    *tb = tabs(d);
    return d;
  }
  const SMCRT_K Prim<T>* P = Tab<T>::prims(a);
  T dv, l;
  T d = convex_sdf_rate<T>(P, R.first, p, u, &dv, &l);
  T t = tangent_bound<T>(d, dv, l, err);
  if (rule == kSegSubtract) {
    for (int i = 1; i < R.count; ++i) d = tmax(d, -prim_sdf<T, XF>(P, R.first + i, p));
  } else {
    for (int i = 1; i < R.count; ++i) {
      const T di = convex_sdf_rate<T>(P, R.first + i, p, u, &dv, &l);
      const T ti = tangent_bound<T>(di, dv, l, err);
      if (rule == kSegUnion) {
        d = tmin(d, di);
        t = tmin(t, ti);
      } else {
        d = tmax(d, di);
        t = tmax(t, ti);
      }
    }
  }
  *tb = d > T(0) ? tmax(d, t) : tabs(d);
  return d;
}

// the way along u out of the simulation volume
template <typename T>
__device__ __forceinline__ T volume_exit(ScP sc, V3<T> p, V3<T> u) {
  const V3<T> c = Tab<T>::bb_c(sc), h = Tab<T>::bb_h(sc);
  const T pv[3] = {p.x, p.y, p.z}, uv[3] = {u.x, u.y, u.z};
  const T cv[3] = {c.x, c.y, c.z}, hv[3] = {h.x, h.y, h.z};
  T t = tinf<T>();
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (uv[i] != T(0)) t = tmin(t, tdiv((uv[i] > T(0) ? cv[i] + hv[i] : cv[i] - hv[i]) - pv[i], uv[i]));
  return t;
}

// ------------------------------------------------------------------ tallies

// A wave's sums, from the escapes on in the order of smcrt_tallies
// (flush_wave).
struct LdsTallies {
  double absorbed[kMaxRegions];
  double sum[9];  // SumSlot
  unsigned long long cnt[15];
};
enum SumSlot { kSEscaped = 0, kSGain = 6, kSLoss, kSStalled };
enum CountSlot {
  kCEvents = 0, kCSteps, kCInteractions, kCInterfaces, kCReflections, kCRefractions, kCCrossings, kCAdvances,
  kCPieces, kCKills, kCStalls, kCEscapes, kCAtomics, kCLaunched
};
constexpr int kTallySums = 9, kTallyCounts = 13;
static_assert(offsetof(smcrt_tallies, events) == 8 * (1 + kTallySums) &&
                  sizeof(smcrt_tallies) == 8 * (1 + kTallySums + kTallyCounts),
              "one lane per entry");

// per-lane run of equal voxels waiting to be added to the grid
struct Run {
  int v;
  double sum;
};

// Grid additions of one wave staged in LDS.  Runs end in the middle of
// divergent DDA loops, a few lanes at a time; staging them and draining the
// stage with every lane active issues the FP64 atomics as full 64-lane
// instructions, which keeps the memory-side atomic units fed steadily.
constexpr int kStage = 256;  // entries per wave
constexpr int kDrain = 64;   // entries that trigger a drain in the walk loop
struct WaveStage {
  double val[kStage];
  int v[kStage];
};

// An interface step of one packet, shared by the lanes of its group (LDS).
// In: position, direction, region; out: surface point in p, normal there in
// u, its cosine with the direction, the ray's way to it, the region across.
constexpr int kSurfaceSlots = 8;  // interface steps a wave takes at a time
struct SurfaceSlot {
  double p[3], u[3], c, t_ray;
  int region, pad;
};

struct Lane {
  Run run;
  WaveStage* stage; // this wave's staging area (LDS)
  double abs_sum;   // absorbed weight not yet added to the workgroup sums
  int abs_region;
  uint32_t n_steps, n_inter;
  // trace
  smcrt_event* rec;
  int n_rec;
};

__device__ __forceinline__ void grid_add(double* F, int v, double val) {
  __builtin_amdgcn_global_atomic_fadd_f64((SMCRT_G double*)F + v, val);
}

// Index of voxel (x, y, z) in a grid of 2x2x2 bricks ((nx+1)/2 by (ny+1)/2
// by (nz+1)/2 bricks, x fastest), a brick's eight voxels consecutive (x
// fastest inside): the neighbours of a path share 64-byte segments, so more
// of a wave's atomic adds travel in one request.
__device__ __forceinline__ int brick_index(int x, int y, int z, int nx, int ny) {
  const int bx = (nx + 1) >> 1, by = (ny + 1) >> 1;
  const int b = ((z >> 1) * by + (y >> 1)) * bx + (x >> 1);
  return (b << 3) | ((z & 1) << 2) | ((y & 1) << 1) | (x & 1);
}

template <typename T>
__device__ __forceinline__ T trcp(T x);
template <>
__device__ __forceinline__ float trcp<float>(float x) { return __builtin_amdgcn_rcpf(x); }
template <>
__device__ __forceinline__ double trcp<double>(double x) { return 1.0 / x; }
// 1/sqrt(x): one instruction (1 ulp) in FP32, correctly rounded in FP64
template <typename T>
__device__ __forceinline__ T trsqrt(T x);
template <>
__device__ __forceinline__ float trsqrt<float>(float x) { return __builtin_amdgcn_rsqf(x); }
template <>
__device__ __forceinline__ double trsqrt<double>(double x) { return 1.0 / __builtin_sqrt(x); }

// One axis of the voxel walk: voxel index, step (+1, -1 or 0), ray
// parameter of the next plane crossing, and the spacing of the crossings.
template <typename T>
struct DdaAxis {
  int i, s;
  T tn, dt;
};

// Narrows [t0, t1] to the part of the ray g + t*gu inside the slab [0, n] of
// one axis (grid units; r = 1/gu).  A ray along the slab (gu = +0, r = inf)
// narrows nothing or, outside it, everything: its products are infinite, and
// the NaN of a ray in one of the faces is taken for that infinity.
template <typename T>
__device__ __forceinline__ void clip_axis(T g, T r, int n, T& t0, T& t1) {
  const T ta = tmax(-g * r, -tinf<T>()), tb = tmin((T(n) - g) * r, tinf<T>());
  t0 = tmax(t0, tmin(ta, tb));
  t1 = tmin(t1, tmax(ta, tb));
}

// The voxel of one axis holding the ray at t0 (on a plane while moving down:
// the voxel below), clamped into the grid, and its next crossing (none, at
// infinity, for a ray along the axis's planes).
template <typename T>
__device__ __forceinline__ DdaAxis<T> start_axis(T g, T gu, T r, int n, T t0) {
  DdaAxis<T> A;
  const T x = g + t0 * gu;
  const bool down = gu < T(0);
  T fl = floor(x);
  fl = down && x == fl ? fl - T(1) : fl;
  fl = tclamp(fl, T(0), T(n - 1));
  A.i = min((int)fl, n - 1);
  A.s = down ? -1 : 1;
  A.tn = tmin(((down ? fl : fl + T(1)) - g) * r, tinf<T>());
  A.dt = tabs(r);
  return A;
}

// Unpolarised Fresnel reflectance between indices n1 -> n2 at incidence
// cosine ci (Sec. 1); *ct receives the transmitted cosine.  Total internal
// reflection gives 1 (and *ct = 0).
__device__ __forceinline__ double fresnel(double n1, double n2, double ci, double* ct) {
  const double eta = n1 / n2;
  const double s2t = eta * eta * (1.0 - ci * ci);
  *ct = 0.0;
  if (s2t >= 1.0) return 1.0;
  const double c2 = __builtin_sqrt(1.0 - s2t);
  const double rs = (n1 * ci - n2 * c2) / (n1 * ci + n2 * c2);
  const double rp = (n1 * c2 - n2 * ci) / (n1 * c2 + n2 * ci);
  *ct = c2;
  return 0.5 * (rs * rs + rp * rp);
}

// ------------------------------------------------------------------ packet

// state of a lane's packet; kDead: the lane has none.  (Held in one vector
// register: as a flag of its own, "has a packet" would be an execution mask
// that every join of the control flow has to patch.)
enum State : int { kTransport = 0, kSurface = 1, kInteract = 2, kDead = 3 };

template <typename T>
struct Packet {
  V3<T> p, u;
  // FP32 only: the part of the position that rounding left out of p
  // (compensated summation of the moves; zero after a jump of position)
  V3<T> pe;
  // remaining optical depth, FP64 in both transport precisions: it is used
  // up over many sphere-tracing steps, and along a grazing path (thousands
  // of steps of delta size) FP32 rounding would let it drift
  double tau;
  T mut, inv_mut;   // of the current region (0 and 0 in ambient)
  double w;
  uint64_t pid;
  uint32_t k;       // event index
  int region;       // n_regions = ambient
  int state;
  int steps;        // sphere-tracing steps in the current event
  T pend;           // straight path along u since the last tally, ending at p
  // previous sphere-tracing step of the current straight segment: surface
  // distance at its start (< 0: none yet) and its length, negated while an
  // over-relaxed step waits for its check at the next evaluation
  T pd, pl;
  // free-flight reuse: radius of a ball about p that holds no surface
  // (< 0: none known) and the interactions taken in it since the distance
  // was evaluated
  T safe;
  int links;
};

constexpr int kReuseLinks = 32;  // interactions per evaluation at most

// A packet still in flight when a resident-serving epoch ends (slot first,
// at the same offset in both precisions, for the host-side kernels that
// sort the records by slot).
template <typename T>
struct SavedPacket {
  int32_t slot;
  int32_t vx[3];
  Packet<T> pk;
};
static_assert(sizeof(SavedPacket<double>) <= kSavedPacketBytes, "saved packet record too large");
static_assert(sizeof(SavedPacket<float>) <= kSavedPacketBytes, "saved packet record too large");

// Writes the live packets of the calling lanes (all lanes of the wave
// active; live lanes save) to the launch's save slab.  The host sizes the
// slab for one packet per lane of every launch of the epoch; a record
// beyond it is counted but not written, and the host fails the epoch.
template <typename T>
__device__ __forceinline__ void save_live(const BatchArgs& B, JobRef a, bool live, const Packet<T>& pk,
                                          const int vx[3], int lane) {
  const uint64_t m = __ballot(live);
  const int n = __popcll(m);
  if (n == 0) return;
  const int leader = __ffsll((unsigned long long)m) - 1;
  unsigned int base = 0;
  if (lane == leader) base = atomicAdd(B.save_count, (unsigned int)n);
  base = __shfl(base, leader);
  if (!live) return;
  const unsigned int i = base + (unsigned int)__popcll(m & ((1ull << lane) - 1ull));
  if (i >= B.save_cap) return;
  SavedPacket<T>* s = reinterpret_cast<SavedPacket<T>*>(static_cast<char*>(B.save) + (size_t)i * kSavedPacketBytes);
  s->slot = a.slot;
  s->vx[0] = vx[0];
  s->vx[1] = vx[1];
  s->vx[2] = vx[2];
  s->pk = pk;
}

// Packet i of job a's resumed packets
template <typename T>
__device__ __forceinline__ void load_saved(JobRef a, unsigned int i, Packet<T>& pk, int vx[3]) {
  const SavedPacket<T>* s =
      reinterpret_cast<const SavedPacket<T>*>(static_cast<const char*>(a.resume) + (size_t)i * kSavedPacketBytes);
  pk = s->pk;
  vx[0] = s->vx[0];
  vx[1] = s->vx[1];
  vx[2] = s->vx[2];
}

// What the walk needs of a packet's own region, in LDS.  Lanes are in
// different regions: read from the scene tables this would be a vector load,
// which waits for every atomic that the wave has issued before it.
template <typename T>
struct RegionRow {
  double mua, mut, n;
  T mut_t, inv_mut_t;
  T hg_b, hg_c, hg_d;
  int iso;
};
template <typename T>
using Regions = const __attribute__((address_space(3))) RegionRow<T>*;

// Fills the table of job a's scene (the ambient slot included) with threads
// t, t + stride, ...
template <typename T>
__device__ __forceinline__ void fill_regions(JobRef a, RegionRow<T>* rows, int t, int stride) {
  ScP sc = kptr(a.sc);
  for (int r = t; r <= sc->n_regions; r += stride) {
    RegRef R = sc->reg[r];
    rows[r] = RegionRow<T>{R.mua, R.mut, R.n, Tab<T>::mut(R), Tab<T>::inv_mut(R), Tab<T>::hg_b(R), Tab<T>::hg_c(R),
                           Tab<T>::hg_d(R), R.iso};
  }
}

template <typename T>
__device__ __forceinline__ void set_region(Regions<T> rg, Packet<T>& pk, int r) {
  pk.region = r;
  pk.mut = rg[r].mut_t;
  pk.inv_mut = rg[r].inv_mut_t;
}

template <typename T, bool TRACE>
__device__ __forceinline__ void record(JobRef a, const Packet<T>& pk, Lane& ln, int type) {
  if constexpr (TRACE) {
    if (ln.n_rec < a.max_records) {
      smcrt_event e;
      e.event = pk.k;
      e.type = (uint32_t)type;
      e.region = pk.region == a.sc->n_regions ? -1 : pk.region;
      e.pad = 0;
      // FP32: the position with its compensation, as the walk carries it
      e.p[0] = (double)pk.p.x + (double)pk.pe.x;
      e.p[1] = (double)pk.p.y + (double)pk.pe.y;
      e.p[2] = (double)pk.p.z + (double)pk.pe.z;
      e.u[0] = pk.u.x; e.u[1] = pk.u.y; e.u[2] = pk.u.z;
      e.w = pk.w;
      e.tau = pk.tau;
      ln.rec[ln.n_rec] = e;
    }
    ++ln.n_rec;
  }
}

// Moves the packet len along u.  The tally is deferred: the straight path
// since the last change of direction collects in pend and is credited to
// the grid in one pass by tally_path, which runs before the direction
// changes or the position jumps (interactions, interface events) and when
// the packet ends.  Collinear sphere-tracing steps thus share one DDA, and
// the lanes of a wave run it together.
//
// In FP32 the position is a compensated sum (2Sum per axis, exact for any
// magnitudes, also where a move is longer than the coordinate near the
// coordinate planes): pe keeps what rounding dropped from p and is added
// back on the next move.  A
// sphere-tracing step that runs nearly parallel to a face a few surface
// thresholds away moves p across that face by far less than p's ulp; a
// plain sum would drop every one of those moves, the packet would slide
// along the face at a fixed depth in steps of that depth, and a walk of
// 0.5 cm would take some 4e4 steps where the FP64 walk takes 2e3.
// s = fl(a + b) and *e = a + b - s exactly (Knuth's 2Sum; six additions,
// no condition on |a| and |b|)
template <typename T>
__device__ __forceinline__ T two_sum(T a, T b, T* e) {
  const T s = a + b;
  const T bb = s - a;
  *e = (a - (s - bb)) + (b - bb);
  return s;
}

// The packet is put at the FP64 point q: in FP32 as the float nearest q
// plus the float nearest the rest, so a re-placement at an interface keeps
// q to about 2^-48 of its size, as the compensated moves do.
template <typename T>
__device__ __forceinline__ void set_position(Packet<T>& pk, V3<double> q) {
  pk.p = from_d<T>(q);
  if constexpr (sizeof(T) == 4) pk.pe = from_d<T>(q - to_d(pk.p));
  else pk.pe = mk(T(0), T(0), T(0));
}

// The move itself: p (+ pe) += len u, compensated in FP32.
template <typename T>
__device__ __forceinline__ void shift(Packet<T>& pk, T len) {
  if constexpr (sizeof(T) == 4) {
    const V3<T> d = len * pk.u + pk.pe;
    V3<T> e;
    pk.p.x = two_sum(pk.p.x, d.x, &e.x);
    pk.p.y = two_sum(pk.p.y, d.y, &e.y);
    pk.p.z = two_sum(pk.p.z, d.z, &e.z);
    pk.pe = e;
  } else {
    pk.p = pk.p + len * pk.u;
  }
}

template <typename T>
__device__ __forceinline__ void advance(Packet<T>& pk, T len) {
  shift(pk, len);
  pk.pend += len;
}

// Sphere-tracing move of len along u (negative: back along u), charged to
// the pending path and the optical depth.  Returns the charged distance.
template <typename T>
__device__ __forceinline__ T step_along(Packet<T>& pk, T len) {
  advance(pk, len);
  pk.tau -= (double)pk.mut * (double)len;
  return len;
}

// What the SDF walk's tally keeps per wave, in scalar registers: entries
// waiting in the stage, and the counts of pieces and of additions issued.
struct WaveTally {
  int n;
  unsigned long long pieces, atomics;
};

// Adds the SDF walk's staged entries to F once at least min_count are waiting.
__device__ __forceinline__ void tally_drain(double* F, WaveStage& S, WaveTally& wt, int min_count, int lane) {
  if (wt.n > 0 && wt.n >= min_count) {
    for (int i = lane; i < wt.n; i += 64) grid_add(F, S.v[i], S.val[i]);
    wt.n = 0;
  }
}

// c ? a : b of values (between variables of an enclosing scope the operator
// picks one of their addresses, which keeps them in memory)
__device__ __forceinline__ int pick(bool c, int a, int b) { return c ? a : b; }

// Adds val at voxel v to the lane's run, for the lanes with some set: a run
// that v ends is staged, or added to F where the stage is full.  SAME: v may
// be the run's own voxel.  Called with every lane of the wave active.
template <bool SAME>
__device__ __forceinline__ void run_piece(double* F, WaveStage& S, WaveTally& wt, Run& run, bool some, int v, double val) {
  const bool same = SAME && v == run.v;
  const bool push = some && !same && run.v >= 0;
  const uint64_t ends = __ballot(push);
  if (ends != 0ull) {
    const int n = __popcll(ends);
    if (wt.n + n <= kStage) {
      const int at = wt.n + __builtin_amdgcn_mbcnt_hi((uint32_t)(ends >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ends, 0u));
      if (push) {
        S.v[at] = run.v;
        S.val[at] = run.sum;
      }
      wt.n += n;
    } else if (push) {
      grid_add(F, run.v, run.sum);
    }
    wt.atomics += (unsigned long long)n;
  }
  wt.pieces += (unsigned long long)__popcll(__ballot(some));
  const double sum = same ? run.sum + val : val;
  run.sum = some ? sum : run.sum;
  run.v = some ? v : run.v;
}

// The pieces of the lanes' paths, from t to t1.  A crossing is some forty
// vector instructions, and what bounds the tally is the wave's wait for its
// longest path, so the loop is one straight body for all lanes: no lane mask
// but a flag, the axes in named registers, the voxel index stepped by the axis
// stride, and the number of staged entries in a scalar register (ends of runs
// take their places in the stage by a ballot; read from LDS at each run, it
// was a chain of two LDS accesses per piece).  Consecutive pieces of one path
// are in different voxels: only the first can continue the lane's run.  (With
// the walk's steps in one straight body too: 64 runs of 1e5 packets in a batch
// 7 % less time, 1e4 packets of the vessel scene and 1e5 of the 50^3 sphere
// 16 %; 1e7 of the slab, bound by the additions themselves, the same.)
template <typename T, bool BRICK>
__device__ __forceinline__ void tally_pieces(double* F, WaveStage& S, WaveTally& wt, Run& run, bool active, int lin,
                                             DdaAxis<T> X, DdaAxis<T> Y, DdaAxis<T> Z, int nx, int ny, int nz, T t, T t1,
                                             double w) {
  // steps left on each axis before the path is off the grid
  int rx = X.s > 0 ? nx - 1 - X.i : X.i, ry = Y.s > 0 ? ny - 1 - Y.i : Y.i, rz = Z.s > 0 ? nz - 1 - Z.i : Z.i;
  // index steps; bricks: inside the brick, and across its face (a step is
  // inside when the index bit of the axis is clear moving up, set moving down)
  const int by_n = (ny + 1) >> 1, bx_n = (nx + 1) >> 1;
  const int ix = X.s, iy = BRICK ? Y.s * 2 : Y.s * nx, iz = BRICK ? Z.s * 4 : Z.s * (nx * ny);
  const int ox = X.s * 7, oy = Y.s * (8 * bx_n - 2), oz = Z.s * (8 * bx_n * by_n - 4);
  const int down = (X.s < 0 ? 1 : 0) | (Y.s < 0 ? 2 : 0) | (Z.s < 0 ? 4 : 0);
  auto piece = [&](bool first) __attribute__((always_inline)) {
    const T m = tmin(X.tn, tmin(Y.tn, Z.tn)), tn = tmin(m, t1);
    const T len = tn - t;
    const double val = w * (double)len;
    if (first) run_piece<true>(F, S, wt, run, active && len > T(0), lin, val);
    else run_piece<false>(F, S, wt, run, active && len > T(0), lin, val);
    // cross the nearest plane (ties: x before y before z)
    const bool bx = X.tn == m, by = !bx && Y.tn == m, bz = !bx && !by;
    int step = pick(bx, ix, pick(by, iy, iz));
    if constexpr (BRICK) {
      const int out = pick(bx, ox, pick(by, oy, oz)), bit = bx ? 1 : (by ? 2 : 4);
      step = pick(((lin ^ down) & bit) != 0, out, step);
    }
    lin += step;
    X.tn = bx ? X.tn + X.dt : X.tn;
    Y.tn = by ? Y.tn + Y.dt : Y.tn;
    Z.tn = bz ? Z.tn + Z.dt : Z.tn;
    rx -= bx ? 1 : 0;
    ry -= by ? 1 : 0;
    rz -= bz ? 1 : 0;
    t = tn;
    active = active && tn < t1 && (rx | ry | rz) >= 0;
  };
  piece(true);
  while (__ballot(active) != 0ull) piece(false);
}

// Path-length estimator (Sec. 3.1): weight * length of the packet's pending
// straight path, which ends at its position, credited to every voxel it
// crosses, by a 3-D DDA in voxel units.  Voxel i spans [lo + i*D, lo +
// (i+1)*D); indices are clamped on entry and the walk stops when it steps off
// the grid.  Called with every lane of the wave active; the lanes with want
// set credit their paths together.
template <typename T>
__device__ __forceinline__ void tally_path(JobRef a, const Packet<T>& pk, bool want, Lane& ln, WaveTally& wt) {
  if (a.fluence == nullptr || __ballot(want) == 0ull) return;
  ScP sc = fresh(kptr(a.sc));
  const int nx = sc->g_dims[0], ny = sc->g_dims[1], nz = sc->g_dims[2];
  // One straight block, the lanes' conditions selected: nested branches cost
  // an exec mask and the zeros of some fourteen results each.  (1e3 packets of
  // the 50^3 sphere 11 % less time, 64 runs of 1e5 5 %, 1e6 of the cylinder and
  // 2e5 of the gallery 4 %, 1e7 of the slab 1 %.)
  const V3<T> inv = Tab<T>::g_inv(sc);
  const V3<T> lo = Tab<T>::g_lo(sc);
  const T len = pk.pend;
  const V3<T> u = pk.u, p = pk.p - len * u;
  T gx = (p.x - lo.x) * inv.x, gy = (p.y - lo.y) * inv.y, gz = (p.z - lo.z) * inv.z;
  T ux = u.x * inv.x + T(0), uy = u.y * inv.y + T(0), uz = u.z * inv.z + T(0);  // (no -0)
  hold(gx);
  hold(gy);
  hold(gz);
  hold(ux);
  hold(uy);
  hold(uz);
  const T rx = trcp(ux), ry = trcp(uy), rz = trcp(uz);
  T t0 = T(0), t1 = len;
  clip_axis(gx, rx, nx, t0, t1);
  clip_axis(gy, ry, ny, t0, t1);
  clip_axis(gz, rz, nz, t0, t1);
  const bool active = want && __builtin_isfinite(gx + gy + gz + ux + uy + uz + len) && t1 > t0;
  const DdaAxis<T> X = start_axis(gx, ux, rx, nx, t0), Y = start_axis(gy, uy, ry, ny, t0),
                   Z = start_axis(gz, uz, rz, nz, t0);
  if (a.brick)
    tally_pieces<T, true>(a.fluence, *ln.stage, wt, ln.run, active, brick_index(X.i, Y.i, Z.i, nx, ny), X, Y, Z, nx, ny, nz,
                          t0, t1, pk.w);
  else
    tally_pieces<T, false>(a.fluence, *ln.stage, wt, ln.run, active, X.i + nx * (Y.i + ny * Z.i), X, Y, Z, nx, ny, nz, t0,
                           t1, pk.w);
}

// Escape image (Sec. 3.2 and Sec. 5: the light at a single plane of
// interest).  A packet leaving through the detector face adds its weight to
// the pixel holding the point where its straight path crosses the face's
// plane: traced back along u from its position when that lies beyond the
// plane and the packet moves outward, else its position.  The axis is a
// template argument: selecting a packet coordinate by a run-time axis lets
// the compiler index the packet in memory, which moves it to scratch.
template <int AX, typename T>
__device__ __forceinline__ void detect_on(JobRef a, ScP sc, V3<T> p, V3<T> u, double w, T sg, T plane) {
  const T pa = AX == 0 ? p.x : (AX == 1 ? p.y : p.z);
  const T ua = AX == 0 ? u.x : (AX == 1 ? u.y : u.z);
  const T over = (pa - plane) * sg, out = ua * sg;
  if (over > T(0) && out > T(0)) p = p - (over / out) * u;
  const T c1 = AX == 0 ? p.y : p.x, c2 = AX == 2 ? p.y : p.z;
  const T x = (c1 - (T)sc->det_lo[0]) / ((T)sc->det_hi[0] - (T)sc->det_lo[0]) * (T)sc->det_dims[0];
  const T y = (c2 - (T)sc->det_lo[1]) / ((T)sc->det_hi[1] - (T)sc->det_lo[1]) * (T)sc->det_dims[1];
  // bounds in floating point, before any conversion (NaN fails too)
  if (!(x >= T(0) && y >= T(0) && x < (T)sc->det_dims[0] && y < (T)sc->det_dims[1])) return;
  const int i = (int)floor(x), j = (int)floor(y);
  grid_add(a.detector, i + sc->det_dims[0] * j, w);
}

template <typename T>
__device__ __forceinline__ void detect(JobRef a, const Packet<T>& pk, int face, T plane) {
  if (a.detector == nullptr) return;
  ScP sc = kptr(a.sc);
  if (face != sc->det_face) return;
  const T sg = (face & 1) ? T(1) : T(-1);
  switch (face >> 1) {
    case 0: detect_on<0>(a, sc, pk.p, pk.u, pk.w, sg, plane); break;
    case 1: detect_on<1>(a, sc, pk.p, pk.u, pk.w, sg, plane); break;
    default: detect_on<2>(a, sc, pk.p, pk.u, pk.w, sg, plane); break;
  }
}

__device__ __forceinline__ void add_absorbed(LdsTallies& L, Lane& ln, int r, double dA) {
  if (r != ln.abs_region) {
    if (ln.abs_region >= 0) atomicAdd(&L.absorbed[ln.abs_region], ln.abs_sum);
    ln.abs_region = r;
    ln.abs_sum = 0.0;
  }
  ln.abs_sum += dA;
}

// emission, event 0 (Sec. 3.1 sources; Eq. 1)
template <typename T, bool TRACE, bool XF>
__device__ void emit(JobRef a, Regions<T> rg, Packet<T>& pk, Lane& ln, LdsTallies& L) {
  ScP sc = kptr(a.sc);
  const U4 r = philox10(0u, (uint32_t)pk.pid, (uint32_t)(pk.pid >> 32), 0u, (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
  const T x0 = xi_of<T>(r.w0), x1 = xi_of<T>(r.w1), x3 = xi_of<T>(r.w3);
  const SMCRT_K double* s = sc->src;
  // the emission point in FP64 (the source's place plus the sampled offset)
  V3<double> p = mk(s[0], s[1], s[2]);
  V3<T> u;
  const int kind = sc->src_kind;
  if (kind == kPoint) {
    const T ct = T(2) * x0 - T(1);
    const T st = T(2) * tsqrt(x0 * (T(1) - x0));  // sqrt(1 - ct^2) without cancellation
    T sp, cp;
    tsincos_2pi(x1, &sp, &cp);
    u = mk(st * cp, st * sp, ct);
  } else if (kind == kPencil) {
    u = mk((T)s[3], (T)s[4], (T)s[5]);
  } else if (kind == kDisc) {
    const T rr = (T)s[3] * tsqrt(x0);
    T sp, cp;
    tsincos_2pi(x1, &sp, &cp);
    p = mk(p.x + (double)(rr * cp), p.y + (double)(rr * sp), p.z);
    u = mk((T)s[4], (T)s[5], (T)s[6]);
  } else {
    p = mk(p.x + s[3] * (2.0 * (double)x0 - 1.0), p.y + s[4] * (2.0 * (double)x1 - 1.0), p.z);
    u = mk((T)s[5], (T)s[6], (T)s[7]);
  }
  const T il = T(1) / tsqrt(dot(u, u));
  set_position(pk, p);
  pk.u = il * u;
  pk.w = 1.0;
  pk.tau = (double)(-tlog(x3));
  pk.k = 0;
  pk.steps = 0;
  pk.pd = T(-1);
  pk.pl = T(0);
  pk.safe = T(-1);
  pk.links = 0;
  pk.pend = T(0);
  pk.state = kTransport;
  set_region(rg, pk, region_of<T, XF>(a, pk.p));
  atomicAdd(&L.cnt[kCLaunched], 1ull);
  record<T, TRACE>(a, pk, ln, SMCRT_EV_EMIT);
}

// absorption, Henyey-Greenstein scattering, roulette, next free path.
// Returns false when the packet ends.
template <typename T, bool TRACE>
__device__ bool interact(JobRef a, Regions<T> rg, Packet<T>& pk, Lane& ln, LdsTallies& L) {
  ScP sc = fresh(kptr(a.sc));
  const __attribute__((address_space(3))) RegionRow<T>& R = rg[pk.region];
  pk.k += 1;
  ++ln.n_inter;
  const U4 r = philox10(pk.k, (uint32_t)pk.pid, (uint32_t)(pk.pid >> 32), 0u, (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
  // implicit capture: the fraction mu_a/mu_t of the weight stays here
  const double dA = pk.w * R.mua / R.mut;
  add_absorbed(L, ln, pk.region, dA);
  pk.w -= dA;
  if (pk.w == 0.0) {
    record<T, TRACE>(a, pk, ln, SMCRT_EV_ABSORB);
    return false;
  }
  // scattering angle from the HG inverse CDF; azimuth uniform.  The CDF is
  // inverted for 1 - cos(theta) directly,
  //   1 - cos = (1 - g)(1 - xi)(f + 1 - g) / D,  D = 1 - g + 2 g xi,
  //   f = (1 - g^2) / D,
  // which has no cancellation near forward scattering, so FP32 keeps
  // sin(theta) = sqrt((1 - cos)(1 + cos)) to full relative precision.
  const T x0 = xi_of<T>(r.w0), x1 = xi_of<T>(r.w1);
  T omc;
  if (R.iso) {
    omc = T(2) * (T(1) - x0);
  } else {
    const T D = R.hg_c + R.hg_d * x0;
    const T f = tdiv(R.hg_b, D);
    omc = tdiv(R.hg_c * (T(1) - x0) * (f + R.hg_c), D);
  }
  omc = tclamp(omc, T(0), T(2));
  const T ct = T(1) - omc;
  const T st = tsqrt(omc * (T(2) - omc));
  T sp, cp;
  tsincos_2pi(x1, &sp, &cp);
  const V3<T> u = pk.u;
  V3<T> v;
  if (tabs(u.z) > T(1) - T(1e-5)) {
    v = mk(st * cp, st * sp, (u.z >= T(0) ? ct : -ct));
  } else {
    // sqrt(1 - uz^2) from the other two components: no cancellation near the poles
    const T tt = tsqrt(u.x * u.x + u.y * u.y);
    const T itt = trcp(tt);
    v.x = st * (u.x * u.z * cp - u.y * sp) * itt + u.x * ct;
    v.y = st * (u.y * u.z * cp + u.x * sp) * itt + u.y * ct;
    v.z = -st * cp * tt + u.z * ct;
  }
  pk.u = trsqrt(dot(v, v)) * v;
  // Russian roulette on the weight
  if (pk.w < sc->w_threshold) {
    const double x2 = xi_of<double>(r.w2);
    if (x2 < sc->inv_m) {
      atomicAdd(&L.sum[kSGain], (sc->m_d - 1.0) * pk.w);
      pk.w *= sc->m_d;
    } else {
      atomicAdd(&L.sum[kSLoss], pk.w);
      atomicAdd(&L.cnt[kCKills], 1ull);
      record<T, TRACE>(a, pk, ln, SMCRT_EV_KILL);
      return false;
    }
  }
  pk.tau = (double)(-tlog(xi_of<T>(r.w3)));
  pk.steps = 0;
  pk.pd = T(-1);
  record<T, TRACE>(a, pk, ln, SMCRT_EV_SCATTER);
  return true;
}

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// First job of the launch's geometry, scanning from `start`, whose packet
// counter has not reached its packet count; -1 when every such job is handed
// out.  Wave uniform.
__device__ __forceinline__ int pick_job(const SMCRT_K WalkArgs* jobs, const BatchArgs& B, int start) {
  for (int i = 0; i < B.n_jobs; ++i) {
    const int j = (start + i) % B.n_jobs;
    JobRef J = jobs[j];
    if (J.geometry != B.geometry) continue;
    const unsigned long long c = __hip_atomic_load(J.counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t cu = ((uint64_t)__builtin_amdgcn_readfirstlane((unsigned)(c >> 32)) << 32) |
                        (uint64_t)__builtin_amdgcn_readfirstlane((unsigned)c);
    if (cu < J.n) return j;
    if (J.resume_n > 0) {  // packets of an earlier epoch left to resume
      const unsigned int r = __hip_atomic_load(J.resume_next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__builtin_amdgcn_readfirstlane(r) < J.resume_n) return j;
    }
  }
  return -1;
}

// Copies job a's FP32 capsule records into the workgroup's LDS table (two
// float4 per capsule); false, with nothing copied, when the job has none or
// more than the table holds.  Called by every thread of the workgroup; the
// caller's barrier makes the table visible.
__device__ __forceinline__ bool stage_caps(JobRef a, F4* dst) {
  const SMCRT_K Accel& A = kptr(a.sc)->acc;
  if (A.region < 0 || !A.caps || A.n_prims > kStageCaps || a.acc_capf == nullptr) return false;
  const F4* src = reinterpret_cast<const F4*>(a.acc_capf);
  const int n = 2 * A.n_prims;
  for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = src[i];
  return true;
}

// Called with every lane of the wave active.
__device__ __forceinline__ void clear_tallies(LdsTallies& L, int lane) {
  if (lane < kMaxRegions) L.absorbed[lane] = 0.0;
  else if (lane < kMaxRegions + kTallySums) L.sum[lane - kMaxRegions] = 0.0;
  else if (lane < kMaxRegions + kTallySums + 15) L.cnt[lane - kMaxRegions - kTallySums] = 0ull;
  __threadfence_block();
}

// Adds a wave's pending sums to job a's outputs and clears them.  Called with
// every lane of the wave active.
__device__ __forceinline__ void flush_wave(JobRef a, Lane& ln, WaveTally& wt, LdsTallies& L, int lane) {
  if (a.fluence != nullptr) {
    tally_drain(a.fluence, *ln.stage, wt, 1, lane);
  }
  if (ln.run.v >= 0) {
    grid_add(a.fluence, ln.run.v, ln.run.sum);
    atomicAdd(&L.cnt[kCAtomics], 1ull);
  }
  if (ln.abs_region >= 0) atomicAdd(&L.absorbed[ln.abs_region], ln.abs_sum);
  atomicAdd(&L.cnt[kCSteps], (unsigned long long)ln.n_steps);
  atomicAdd(&L.cnt[kCInteractions], (unsigned long long)ln.n_inter);
  if (lane == 0) {
    L.cnt[kCPieces] += wt.pieces;
    L.cnt[kCAtomics] += wt.atomics;
  }
  wt.pieces = wt.atomics = 0ull;
  ln.run.v = -1;
  ln.run.sum = 0.0;
  ln.abs_region = -1;
  ln.abs_sum = 0.0;
  ln.n_steps = ln.n_inter = 0;
  if (lane == 0) L.cnt[kCEvents] = L.cnt[kCInteractions] + L.cnt[kCInterfaces];
  __threadfence_block();
  // One lane per entry, and none for a zero: waves that found no packet left
  // have only zeros, and the additions of all waves to one cache line queue
  // up behind each other.  (Lane 0 adding every entry in turn: a launch of
  // one packet of the 50^3 sphere 0.36 ms more, of 1e3 0.26.)
  if (a.absorbed != nullptr && lane < a.sc->n_regions && L.absorbed[lane] != 0.0)
    unsafeAtomicAdd(a.absorbed + lane, L.absorbed[lane]);
  if (a.tallies != nullptr) {
    double* sums = reinterpret_cast<double*>(a.tallies);
    unsigned long long* counts = reinterpret_cast<unsigned long long*>(sums + 1 + kTallySums);
    const int k = lane - 32;
    if (lane < kTallySums) {
      if (L.sum[lane] != 0.0) unsafeAtomicAdd(sums + 1 + lane, L.sum[lane]);
    } else if (lane == kTallySums) {
      if (L.cnt[kCLaunched] != 0ull) unsafeAtomicAdd(sums, (double)L.cnt[kCLaunched]);
    } else if (k >= 0 && k < kTallyCounts) {
      if (L.cnt[k] != 0ull) atomicAdd(counts + k, L.cnt[k]);
    }
  }
  __threadfence_block();
  clear_tallies(L, lane);
}

}  // namespace smcrt
