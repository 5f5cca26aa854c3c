// accel.hip -- device build of the uniform-grid acceleration of one union
// region (Sec. 5: a space-partitioning structure so that a step need not
// evaluate every SDF of a large collection).
//
// Passes, all on the device:
//   count : every primitive adds 1 to each cell its bounding box, grown by
//           the margin, overlaps;
//   scan  : the counts become CSR offsets (sums of tiles, then each tile);
//   fill  : every primitive writes its index into those cells' lists;
// then the ring distances of the empty cells, one axis after the other.
// count and fill share one cell-range routine, so they agree exactly; fill
// still checks every write against the capacity the host allocated.
// A workgroup shares one primitive's cells: a 2000-capsule network has long
// capsules of thousands of cells, which one thread each walked in 1.2 (count)
// and 1.6 ms (fill) with 8 workgroups on the chip.  With that, a scan by one
// workgroup (0.43 ms) and 15 relaxation passes for the rings (0.10 ms), a
// 64^3 build took 3.4 ms; as here it takes 0.07 ms.
#include <hip/hip_runtime.h>

#include "launch.h"
#include "layout.h"

namespace smcrt {

// inclusive cell range [c0, c1] of a primitive's world box (packed by the
// host for every kind, placement and modifier) grown by the margin, clamped
__device__ __forceinline__ void cell_range(const Accel& A, const PrimD& P, int c0[3], int c1[3]) {
  for (int i = 0; i < 3; ++i) {
    const double a = (P.box_lo[i] - A.margin - A.lo[i]) * A.inv_cell[i];
    const double b = (P.box_hi[i] + A.margin - A.lo[i]) * A.inv_cell[i];
    int x0 = (int)floor(fmax(a, -1.0)), x1 = (int)floor(fmin(b, (double)A.dims[i]));
    x0 = x0 < 0 ? 0 : (x0 >= A.dims[i] ? A.dims[i] - 1 : x0);
    x1 = x1 < 0 ? 0 : (x1 >= A.dims[i] ? A.dims[i] - 1 : x1);
    c0[i] = x0;
    c1[i] = x1;
  }
}

// Whether cell (x, y, z) lists the primitive.  A primitive whose box grown
// by the margin overlaps the cell is listed, except a plain capsule whose
// axis segment lies farther than r + margin + (half the cell diagonal) from
// the cell centre: every point of the cell is then more than margin from
// its surface, so a query there never needs it.  The test errs towards
// listing (a relative slack of 1e-9 covers the rounding of the distance).
__device__ __forceinline__ bool cell_lists(const Accel& A, const PrimD& P, int x, int y, int z) {
  if (P.kind != kCapsule || P.flags != 0) return true;
  double c[3], hd2 = 0.0;
  const int ix[3] = {x, y, z};
  for (int i = 0; i < 3; ++i) {
    const double w = 1.0 / A.inv_cell[i];
    c[i] = A.lo[i] + (ix[i] + 0.5) * w - P.v[i];  // cell centre relative to the segment start
    hd2 += 0.25 * w * w;
  }
  const double t = fmin(fmax((c[0] * P.v[3] + c[1] * P.v[4] + c[2] * P.v[5]) * P.v[6], 0.0), 1.0);
  const double d0 = c[0] - t * P.v[3], d1 = c[1] - t * P.v[4], d2 = c[2] - t * P.v[5];
  const double reach = (P.v[7] + A.margin + sqrt(hd2)) * (1.0 + 1e-9);
  return d0 * d0 + d1 * d1 + d2 * d2 <= reach * reach;
}

constexpr int kBuildBlock = 128;                   // threads per primitive
constexpr int kScanBlock = 256, kScanEach = 8;     // a scan tile: kScanEach rounds of a workgroup
constexpr int kScanTile = kScanBlock * kScanEach;

__global__ void accel_zero(uint32_t* __restrict__ a, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) a[i] = 0u;
}

// f(cell) for every cell that lists primitive P, shared by the workgroup
template <typename F>
__device__ __forceinline__ void listed_cells(const Accel& A, const PrimD& P, F f) {
  int c0[3], c1[3];
  cell_range(A, P, c0, c1);
  const int nx = c1[0] - c0[0] + 1, ny = c1[1] - c0[1] + 1, nz = c1[2] - c0[2] + 1;
  const int n = nx * ny * nz;  // at most the grid's cells
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const int x = c0[0] + i % nx, y = c0[1] + (i / nx) % ny, z = c0[2] + i / (nx * ny);
    if (cell_lists(A, P, x, y, z)) f(x + A.dims[0] * (y + A.dims[1] * z));
  }
}

__global__ void __launch_bounds__(kBuildBlock) accel_count(const SceneHeader* __restrict__ sc, const PrimD* __restrict__ pd,
                                                           uint32_t* __restrict__ counts) {
  const Accel& A = sc->acc;
  for (int p = blockIdx.x; p < A.n_prims; p += gridDim.x)
    listed_cells(A, pd[A.first_prim + p], [&](int c) { atomicAdd(&counts[c], 1u); });
}

// sum of v over the workgroup and, in *before, over the threads below this one
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* before) {
  __shared__ uint32_t part[kScanBlock];
  const int t = threadIdx.x;
  part[t] = v;
  __syncthreads();
  for (int off = 1; off < kScanBlock; off <<= 1) {  // Hillis-Steele inclusive scan
    const uint32_t w = t >= off ? part[t - off] : 0u;
    __syncthreads();
    part[t] += w;
    __syncthreads();
  }
  *before = t ? part[t - 1] : 0u;
  const uint32_t all = part[kScanBlock - 1];
  __syncthreads();
  return all;
}

// The cells are cut into tiles of kScanBlock * kScanEach.  sums[tile]: its count
__global__ void __launch_bounds__(kScanBlock) accel_tile_sums(const uint32_t* __restrict__ counts, int n,
                                                              uint32_t* __restrict__ sums) {
  const int base = blockIdx.x * kScanTile;
  uint32_t s = 0, before;
  for (int k = 0; k < kScanEach; ++k) {
    const int i = base + k * kScanBlock + threadIdx.x;
    if (i < n) s += counts[i];
  }
  s = block_scan(s, &before);
  if (threadIdx.x == 0) sums[blockIdx.x] = s;
}

// offsets[0..n]: the tiles' sums before this one, then the scan of the tile
__global__ void __launch_bounds__(kScanBlock) accel_offsets(const uint32_t* __restrict__ counts, int n,
                                                            const uint32_t* __restrict__ sums,
                                                            uint32_t* __restrict__ offsets) {
  const int base = blockIdx.x * kScanTile;
  uint32_t s = 0, before;
  for (int i = threadIdx.x; i < (int)blockIdx.x; i += kScanBlock) s += sums[i];
  uint32_t run = block_scan(s, &before);
  for (int k = 0; k < kScanEach; ++k) {
    const int i = base + k * kScanBlock + threadIdx.x;
    const uint32_t all = block_scan(i < n ? counts[i] : 0u, &before);
    if (i < n) offsets[i] = run + before;
    run += all;
  }
  if (threadIdx.x == 0 && base + kScanTile >= n) offsets[n] = run;
}

__global__ void __launch_bounds__(kBuildBlock) accel_fill(const SceneHeader* __restrict__ sc, const PrimD* __restrict__ pd,
                                                          const uint32_t* __restrict__ offsets,
                                                          uint32_t* __restrict__ cursors, uint32_t* __restrict__ ids) {
  const Accel& A = sc->acc;
  for (int p = blockIdx.x; p < A.n_prims; p += gridDim.x)
    listed_cells(A, pd[A.first_prim + p], [&](int c) {
      const uint64_t slot = (uint64_t)offsets[c] + atomicAdd(&cursors[c], 1u);
      if (slot < A.capacity) ids[slot] = (uint32_t)(A.first_prim + p);
    });
}

// Ring distances: the Chebyshev distance to the nearest cell that lists a
// primitive, kRingMax at most.  The largest of three coordinate distances is
// minimised one axis at a time: along x the distance to the nearest listing
// cell of the row, then along y (z) the smallest of max(way, value there).
// The first axis reads counts, the others the previous axis's distances.
template <int AXIS>
__global__ void __launch_bounds__(256) accel_ring(const SceneHeader* __restrict__ sc, const uint32_t* __restrict__ in,
                                                  uint32_t* __restrict__ out) {
  const Accel& A = sc->acc;
  const int dx = A.dims[0], dy = A.dims[1], n = A.n_cells;
  const int len = A.dims[AXIS], stride = AXIS == 0 ? 1 : (AXIS == 1 ? dx : dx * dy);
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int at = AXIS == 0 ? i % dx : (AXIS == 1 ? (i / dx) % dy : i / (dx * dy));
    auto value = [&](int j) -> uint32_t {
      const uint32_t v = in[i + (j - at) * stride];
      return AXIS == 0 ? (v ? 0u : (uint32_t)kRingMax) : v;
    };
    uint32_t m = value(at);
    for (uint32_t r = 1; r < m; ++r) {  // cells r away are no use once m <= r
      if (at >= (int)r) {
        const uint32_t v = value(at - (int)r);
        m = min(m, max(r, v));
      }
      if (at + (int)r < len) {
        const uint32_t v = value(at + (int)r);
        m = min(m, max(r, v));
      }
    }
    out[i] = m;
  }
}

hipError_t launch_accel_build(const SceneHeader* d_sc, const PrimD* d_pd, int n_prims, int n_cells, uint32_t* counts,
                              uint32_t* cursors, uint32_t* offsets, uint32_t* ids, hipStream_t stream) {
  if (!d_sc || !d_pd || !counts || !cursors || !offsets || !ids || n_prims < 1 || n_cells < 1) return hipErrorInvalidValue;
  const int zb = (n_cells + 255) / 256, cb = zb < 4096 ? zb : 4096;
  const int pb = n_prims < 65536 ? n_prims : 65536, tiles = (n_cells + kScanTile - 1) / kScanTile;
  hipLaunchKernelGGL(accel_zero, dim3(cb), dim3(256), 0, stream, counts, n_cells);
  hipLaunchKernelGGL(accel_count, dim3(pb), dim3(kBuildBlock), 0, stream, d_sc, d_pd, counts);
  // the cursors' place first holds the tiles' sums (fewer than cells)
  hipLaunchKernelGGL(accel_tile_sums, dim3(tiles), dim3(kScanBlock), 0, stream, counts, n_cells, cursors);
  hipLaunchKernelGGL(accel_offsets, dim3(tiles), dim3(kScanBlock), 0, stream, counts, n_cells, cursors, offsets);
  hipLaunchKernelGGL(accel_zero, dim3(cb), dim3(256), 0, stream, cursors, n_cells);
  hipLaunchKernelGGL(accel_fill, dim3(pb), dim3(kBuildBlock), 0, stream, d_sc, d_pd, offsets, cursors, ids);
  // counts and cursors are free after the first axis: ring distances, ending in cursors
  hipLaunchKernelGGL(accel_ring<0>, dim3(cb), dim3(256), 0, stream, d_sc, counts, cursors);
  hipLaunchKernelGGL(accel_ring<1>, dim3(cb), dim3(256), 0, stream, d_sc, cursors, counts);
  hipLaunchKernelGGL(accel_ring<2>, dim3(cb), dim3(256), 0, stream, d_sc, counts, cursors);
  return hipGetLastError();
}

}  // namespace smcrt
