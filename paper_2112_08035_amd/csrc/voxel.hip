// voxel.hip -- voxelisation of an SDF scene onto its fluence grid, the
// geometry of the voxelised comparison model (Sec. 3): each voxel takes the
// region that owns its centre (the highest-index region whose SDF is
// negative there, else the ambient slot), evaluated in FP64 through the same
// region SDFs, uniform-grid acceleration included, that the SDF walk uses;
// and point queries of those SDFs.
#include <hip/hip_runtime.h>

#include "launch.h"
#include "walk_common.h"

namespace smcrt {

__global__ void __launch_bounds__(256) voxelize_kernel(const WalkArgs* __restrict__ job_table, int job,
                                                       uint8_t* __restrict__ vox, size_t n) {
  JobRef a = kptr(job_table)[job];
  ScP sc = kptr(a.sc);
  const int nx = sc->g_dims[0], ny = sc->g_dims[1];
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int ix = (int)(i % (size_t)nx);
    const size_t r = i / (size_t)nx;
    const int iy = (int)(r % (size_t)ny);
    const int iz = (int)(r / (size_t)ny);
    const V3<double> c = mk(sc->g_lo[0] + (ix + 0.5) * sc->g_d[0], sc->g_lo[1] + (iy + 0.5) * sc->g_d[1],
                            sc->g_lo[2] + (iz + 0.5) * sc->g_d[2]);
    vox[i] = (uint8_t)region_of<double, true>(a, c);
  }
}

// The first words of a primitive's record -- kind, flags and shape -- in
// scalar registers, laid out like an evaluation record's.
typedef uint32_t U16p __attribute__((ext_vector_type(16), aligned(4)));
typedef uint32_t U4p __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ StepV<float> load_shape(const SMCRT_K Prim<float>* P) {
  return {*reinterpret_cast<const SMCRT_K U16p*>(P)};
}
__device__ __forceinline__ StepV<double> load_shape(const SMCRT_K Prim<double>* P) {
  const U4p t = *reinterpret_cast<const SMCRT_K U4p*>(reinterpret_cast<const SMCRT_K U16p*>(P) + 1);
  return {*reinterpret_cast<const SMCRT_K U16p*>(P),
          __builtin_shufflevector(t, t, 0, 1, 2, 3, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1)};
}

// region_sdf at N points at once, the next primitive's record on its way
// while this one is worked on.  INLINE: placed primitives inline (where a
// kernel does more than this, that costs it registers, and with them waves).
template <typename T, int N, bool INLINE>
__device__ __forceinline__ void region_sdf_n(JobRef a, RegRef R, const V3<T> (&p)[N], T (&d)[N]) {
  const SMCRT_K Prim<T>* P = Tab<T>::prims(a);
  const int first = R.first, count = R.count, op = R.op;
  StepV<T> cur = load_shape(P + first);
  for (int i = 0;; ++i) {
    const bool more = i + 1 < count;
    const StepV<T> next = load_shape(P + first + (more ? i + 1 : 0));
    const int kind = cur.bits();
    T b[N];
    if (cur.index() != 0) {
#pragma unroll
      for (int k = 0; k < N; ++k) {
        if constexpr (INLINE) b[k] = placed_prim<T>(P, first + i, p[k]);
        else b[k] = placed_prim_sdf<T, true>(P, first + i, p[k]);
      }
    } else if (kind == kCapsule) {
#pragma unroll
      for (int k = 0; k < N; ++k) b[k] = shape_of<T>(kCapsule, cur, p[k]);
    } else {
#pragma unroll
      for (int k = 0; k < N; ++k) b[k] = shape_of<T>(kind, cur, p[k]);
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
      if (i == 0) {
        d[k] = b[k];
      } else if (op == kUnion) {
        d[k] = tmin(d[k], b[k]);
      } else if (op == kSmoothUnion) {
        d[k] = smooth_min(d[k], b[k], Tab<T>::k(R), Tab<T>::inv_k(R));
      } else {
        d[k] = tmax(d[k], op == kSubtract ? -b[k] : b[k]);
      }
    }
    if (!more) return;
    cur = next;
  }
}

// Point queries: every region's SDF at each point (through the uniform grid
// for the accelerated region when accelerated), the point's owner by the
// walk's rule, in transport type T; and, when asked, every region's unit
// normal by the interface step's FP64 central differences (step h_normal).
//
// What bounds it is the evaluations, one primitive after the other: 1e5
// points of the 2000-capsule vessel scene are 1.4e9 capsule distances, and a
// wave waits for the scalar loads of each.  The two offset points of an axis
// share the loads and fill each other's latencies.
//
// kNormalsSplit: a workgroup takes 64 points; its first wave evaluates at the
// points, three others take an axis each, and the normals come together
// through LDS.  kNormals: a lane does all of its point, for launches that
// fill the card so (two waves per SIMD).  With a lane doing one evaluation
// after the other, each waiting for its own loads, the vessel scene's FP64
// distances and normals took, in ms, 7.56 (1e3 points), 7.59 (1e5) and 14.9
// (3e5); split 0.88, 2.5 and 7.0; with kNormals 2.9, 3.5 and 7.0.
// kNormalsSingly: one evaluation after the other, the distances of all regions
// first.  Placed primitives share no loads between two points, and the pair's
// registers cost a wave per SIMD: 1e6 points of the gallery scene 0.297 so,
// 0.307 with kNormals, 0.335 split.  Where no region has a second primitive,
// none is read ahead: 1e6 points of the 50^3 sphere 0.029 so, 0.031 with
// kNormals, 0.043 split, of the three-layer slab 0.064, 0.071 and 0.076.
enum PointsMode { kDistances, kNormals, kNormalsSingly, kNormalsSplit };

// region r at x + h and x - h on the given axis: the difference
__device__ __forceinline__ double axis_difference(JobRef a, int r, bool grid, int axis, V3<double> x, double h) {
  ScP sc = kptr(a.sc);
  const double hx = axis == 0 ? h : 0.0, hy = axis == 1 ? h : 0.0, hz = axis == 2 ? h : 0.0;
  const V3<double> p[2] = {mk(x.x + hx, x.y + hy, x.z + hz), mk(x.x - hx, x.y - hy, x.z - hz)};
  double d[2];
  if (grid) {
#pragma unroll 1
    for (int k = 0; k < 2; ++k) d[k] = accel_sdf<double, true>(a, grid_of<double>(sc->acc), k ? p[1] : p[0]);
  } else {
    region_sdf_n<double, 2, false>(a, sc->reg[r], p, d);
  }
  return d[0] - d[1];
}

__device__ __forceinline__ void store_normal(double* o, double gx, double gy, double gz) {
  V3<double> g = mk(gx, gy, gz);
  g = (1.0 / __builtin_sqrt(dot(g, g))) * g;
  o[0] = g.x;
  o[1] = g.y;
  o[2] = g.z;
}

template <typename T, PointsMode MODE>
__global__ void __launch_bounds__(256)
distance_kernel(const WalkArgs* __restrict__ job_table, int job, const double* __restrict__ pts, uint64_t n,
                int accelerated, double* __restrict__ dist, int32_t* __restrict__ owner, double* __restrict__ normals) {
  constexpr bool kSplit = MODE == kNormalsSplit;
  JobRef a = kptr(job_table)[job];
  ScP sc = kptr(a.sc);
  const int nr = sc->n_regions;
  const double h = sc->h_normal;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const uint64_t batch = kSplit ? 64u : blockDim.x;
  __shared__ double diff[2][3][kSplit ? 64 : 1];  // by region parity: one barrier a region
  for (uint64_t i0 = (uint64_t)blockIdx.x * batch; i0 < n; i0 += (uint64_t)gridDim.x * batch) {
    const uint64_t i = i0 + (kSplit ? lane : (int)threadIdx.x);
    const uint64_t at = i < n ? i : n - 1;
    const V3<double> q = mk(pts[3 * at], pts[3 * at + 1], pts[3 * at + 2]);
    int own = nr;
    for (int r = 0; r < nr; ++r) {
      const bool grid = accelerated && r == a.acc_region;
      double* out = normals + 3 * (i * (uint64_t)nr + r);
      if (!kSplit || wave == 0) {
        const V3<T> p[1] = {mk((T)q.x, (T)q.y, (T)q.z)};
        T d[1];
        if (grid) d[0] = accel_sdf<T, true>(a, grid_of<T>(sc->acc), p[0]);
        else if constexpr (MODE == kNormalsSingly) d[0] = region_sdf<T, true>(a, sc->reg[r], p[0]);
        else region_sdf_n<T, 1, MODE == kDistances>(a, sc->reg[r], p, d);
        if (i < n) dist[i * (uint64_t)nr + r] = (double)d[0];
        if (d[0] < T(0)) own = r;
      }
      if constexpr (MODE == kNormals) {
        double g[3];
#pragma unroll 1
        for (int ax = 0; ax < 3; ++ax) {
          const double v = axis_difference(a, r, grid, ax, q, h);
          if (ax == 0) g[0] = v;
          else if (ax == 1) g[1] = v;
          else g[2] = v;
        }
        if (i < n) store_normal(out, g[0], g[1], g[2]);
      } else if constexpr (kSplit) {
        if (wave != 0) diff[r & 1][wave - 1][lane] = axis_difference(a, r, grid, wave - 1, q, h);
        __syncthreads();
        if (wave == 0 && i < n) store_normal(out, diff[r & 1][0][lane], diff[r & 1][1][lane], diff[r & 1][2][lane]);
      }
    }
    if (owner && i < n && (!kSplit || wave == 0)) owner[i] = own;
    if constexpr (MODE == kNormalsSingly) {
      for (int r = 0; r < nr; ++r) {
        const bool grid = accelerated && r == a.acc_region;
        auto f = [&](double x, double y, double z) {
          return grid ? accel_sdf<double, true>(a, grid_of<double>(sc->acc), mk(x, y, z))
                      : region_sdf<double, true>(a, sc->reg[r], mk(x, y, z));
        };
        if (i < n)
          store_normal(normals + 3 * (i * (uint64_t)nr + r), f(q.x + h, q.y, q.z) - f(q.x - h, q.y, q.z),
                       f(q.x, q.y + h, q.z) - f(q.x, q.y - h, q.z), f(q.x, q.y, q.z + h) - f(q.x, q.y, q.z - h));
      }
    }
    if constexpr (kSplit) __syncthreads();
  }
}

template <typename T>
static void launch_distance_kernel(const WalkArgs* d_jobs, int job, const double* points, uint64_t n, int accelerated,
                                   bool singly, double* dist, int32_t* owner, double* normals, hipStream_t stream) {
  // two waves per SIMD with a point per lane.  us split and not, at 1e5, 2e5
  // and 1e6 points: gallery 49 and 63, 76 and 81, 273 and 262; 20 capsules 53
  // and 66, 75 and 84, 234 and 239; slab 21.6 and 22.7, 27.5 and 25.6, 75 and 64
  constexpr uint64_t kSplitBelow = 131072;
  const bool split = normals && n < kSplitBelow;
  uint64_t blocks = split ? (n + 63) / 64 : (n + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  auto k = distance_kernel<T, kDistances>;
  if (normals) k = split ? distance_kernel<T, kNormalsSplit> : (singly ? distance_kernel<T, kNormalsSingly> : distance_kernel<T, kNormals>);
  hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(256), 0, stream, d_jobs, job, points, n, accelerated, dist, owner,
                     normals);
}

hipError_t launch_distance(int precision, const WalkArgs* d_jobs, int job, const double* points, uint64_t n, int accelerated,
                           bool singly, double* dist, int32_t* owner, double* normals, hipStream_t stream) {
  if (!d_jobs || !points || !dist || job < 0 || n == 0) return hipErrorInvalidValue;
  if (precision == 1) launch_distance_kernel<double>(d_jobs, job, points, n, accelerated, singly, dist, owner, normals, stream);
  else launch_distance_kernel<float>(d_jobs, job, points, n, accelerated, singly, dist, owner, normals, stream);
  return hipGetLastError();
}

hipError_t launch_voxelize(const WalkArgs* d_jobs, int job, uint8_t* vox, size_t n_vox, hipStream_t stream) {
  if (!d_jobs || !vox || job < 0 || n_vox == 0) return hipErrorInvalidValue;
  size_t blocks = (n_vox + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(voxelize_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, d_jobs, job, vox, n_vox);
  return hipGetLastError();
}

}  // namespace smcrt
