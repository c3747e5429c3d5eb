// Discrete gradient paths on a parameter-space map of the metric.
//
// Results: the metric of one transform family (translation, rotation or
// scale) is mapped over a 3D grid of its parameters, and the paths a
// gradient method follows on that map show which starting points reach the
// known optimum; Discussion: that capture range is what separates the
// entropies.  On the grid a path steps from a point to the 26-connected
// neighbour of steepest rise of sign * f,
//   slope = (sign f(q) - sign f(p)) * w,  w = 1, 1/sqrt 2 or 1/sqrt 3
// (the reciprocal of the step length, as the nearest fp64 value), and stops
// at a point no neighbour rises from (a local extremum).  Ties keep the
// first neighbour in (dz, dy, dx) order, each running -1, 0, 1.  NaN points
// are extrema and never entered.  Every point's successor rises strictly, so
// no path revisits a point and each ends within n steps.
#include "paths.h"

#include <stdint.h>

namespace gemi {

namespace {
constexpr double kInvSqrt2 = 0.70710678118654752440;
constexpr double kInvSqrt3 = 0.57735026918962576451;
constexpr int kPathThreads = 256;
constexpr int kSinkThreads = 1024;

unsigned path_grid(int64_t n, int threads, int64_t most) {
  const int64_t g = (n + threads - 1) / threads;
  return (unsigned)(g < most ? (g > 0 ? g : 1) : most);
}
}  // namespace

__global__ __launch_bounds__(kPathThreads) void path_next_kernel(const double* __restrict__ f, int32_t nx,
                                                                 int32_t ny, int32_t nz, double sign,
                                                                 int32_t* __restrict__ next,
                                                                 int64_t* __restrict__ stats) {
  if (blockIdx.x == 0 && threadIdx.x < 4) stats[threadIdx.x] = threadIdx.x == 3 ? INT64_MAX : 0;  // see path_sink_kernel
  const uint32_t n = (uint32_t)nx * (uint32_t)ny * (uint32_t)nz;  // < 2^31
  for (uint32_t p = blockIdx.x * kPathThreads + threadIdx.x; p < n; p += gridDim.x * kPathThreads) {
    const uint32_t r = p / (uint32_t)nx;
    const int32_t x = (int32_t)(p - r * (uint32_t)nx);
    const int32_t z = (int32_t)(r / (uint32_t)ny), y = (int32_t)(r - (uint32_t)z * (uint32_t)ny);
    const double fp = sign * f[p];
    double best = 0.0;
    uint32_t arg = p;
    for (int dz = -1; dz <= 1; ++dz) {
      const int32_t zz = z + dz;
      if (zz < 0 || zz >= nz) continue;
      for (int dy = -1; dy <= 1; ++dy) {
        const int32_t yy = y + dy;
        if (yy < 0 || yy >= ny) continue;
        for (int dx = -1; dx <= 1; ++dx) {
          const int32_t xx = x + dx;
          const int k = (dx != 0) + (dy != 0) + (dz != 0);
          if (xx < 0 || xx >= nx || k == 0) continue;
          const uint32_t q = ((uint32_t)zz * (uint32_t)ny + (uint32_t)yy) * (uint32_t)nx + (uint32_t)xx;
          const double w = k == 1 ? 1.0 : (k == 2 ? kInvSqrt2 : kInvSqrt3);
          const double s = (sign * f[q] - fp) * w;
          if (s > best) {
            best = s;
            arg = q;
          }
        }
      }
    }
    next[p] = (int32_t)arg;
  }
}

// Follows each point's successors to the extremum its path ends at, and
// gathers the map's figures over the points: extrema, points that end where
// the centre does, and the smallest Chebyshev distance from the centre of a
// point that ends elsewhere.  The step bound n is never reached by a strictly
// rising path; it only makes the loops' end independent of the data.
//
// While it runs, stats holds: [0] extrema << 32 | basin (n < 2^31), [1] the
// workgroups done, [3] the distance; the last workgroup replaces them by
//   [0] extrema, [1] sink of the centre, [2] points ending there,
//   [3] capture radius: one less than the nearest point that ends elsewhere,
//   or, when every point ends at the centre's extremum, the grid's largest
//   Chebyshev distance from the centre.
// What bounds it: the chains of dependent loads, and the atomics on one line,
// about 11 ns each, hence few large workgroups and three of them per workgroup
// (a 51^3 map: with three per wave of 256-thread workgroups the figures alone
// took 76 us, with their own launches for start and end 94 us a call; now
// 17).
__global__ __launch_bounds__(kSinkThreads) void path_sink_kernel(const int32_t* __restrict__ next, int32_t nx,
                                                                 int32_t ny, int32_t nz, int32_t cx, int32_t cy,
                                                                 int32_t cz, int32_t* __restrict__ sink,
                                                                 int64_t* __restrict__ stats) {
  const uint32_t n = (uint32_t)nx * (uint32_t)ny * (uint32_t)nz;  // < 2^31
  auto follow = [&](uint32_t p) -> uint32_t {
    for (uint32_t step = 0; step < n; ++step) {
      const uint32_t r = (uint32_t)next[p];
      if (r == p) break;
      p = r;
    }
    return p;
  };
  const uint32_t target = follow(((uint32_t)cz * (uint32_t)ny + (uint32_t)cy) * (uint32_t)nx + (uint32_t)cx);
  uint64_t counts = 0;  // extrema << 32 | basin
  uint32_t dmin = UINT32_MAX;
  for (uint32_t p = blockIdx.x * kSinkThreads + threadIdx.x; p < n; p += gridDim.x * kSinkThreads) {
    const uint32_t q = follow(p);
    sink[p] = (int32_t)q;
    counts += q == p ? 1ull << 32 : 0;
    if (q == target) {
      ++counts;
    } else {
      const uint32_t r = p / (uint32_t)nx;
      const int32_t x = (int32_t)(p - r * (uint32_t)nx);
      const int32_t z = (int32_t)(r / (uint32_t)ny), y = (int32_t)(r - (uint32_t)z * (uint32_t)ny);
      const uint32_t d = (uint32_t)max(abs(x - cx), max(abs(y - cy), abs(z - cz)));
      dmin = d < dmin ? d : dmin;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    counts += __shfl_xor(counts, off, 64);
    const uint32_t o = __shfl_xor(dmin, off, 64);
    dmin = o < dmin ? o : dmin;
  }
  __shared__ uint64_t wave_counts[kSinkThreads / 64];
  __shared__ uint32_t wave_dmin[kSinkThreads / 64];
  if ((threadIdx.x & 63) == 0) {
    wave_counts[threadIdx.x >> 6] = counts;
    wave_dmin[threadIdx.x >> 6] = dmin;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int w = 1; w < kSinkThreads / 64; ++w) {
    counts += wave_counts[w];
    dmin = wave_dmin[w] < dmin ? wave_dmin[w] : dmin;
  }
  uint64_t* st = (uint64_t*)stats;
  if (counts) __hip_atomic_fetch_add(&st[0], counts, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (dmin != UINT32_MAX) __hip_atomic_fetch_min(&st[3], (uint64_t)dmin, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // Both are done before the ticket: while the kernel runs stats is accessed by
  // agent-scope atomics alone, which on gfx950 are coherent over the XCDs, and
  // vmcnt(0) waits until they are done.  (Fences would write back and invalidate the L2s
  // as well: a 101^3 map 69.7 -> 75.3 us.)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (__hip_atomic_fetch_add(&st[1], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != gridDim.x - 1) return;
  asm volatile("" ::: "memory");
  const uint64_t all = __hip_atomic_load(&st[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t near = __hip_atomic_load(&st[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int32_t ex = max(cx, nx - 1 - cx), ey = max(cy, ny - 1 - cy), ez = max(cz, nz - 1 - cz);
  stats[0] = (int64_t)(all >> 32);
  stats[1] = target;
  stats[2] = (int64_t)(all & 0xFFFFFFFFull);
  stats[3] = near == (uint64_t)INT64_MAX ? max(ex, max(ey, ez)) : (int64_t)near - 1;
}

hipError_t launch_map_paths(const PathsLaunch& L, hipStream_t s) {
  const int64_t n = (int64_t)L.nx * L.ny * L.nz;
  hipLaunchKernelGGL(path_next_kernel, dim3(path_grid(n, kPathThreads, 8192)), dim3(kPathThreads), 0, s, L.values, L.nx,
                     L.ny, L.nz, L.sign, L.next, L.stats);
  hipLaunchKernelGGL(path_sink_kernel, dim3(path_grid(n, kSinkThreads, 2048)), dim3(kSinkThreads), 0, s, L.next, L.nx,
                     L.ny, L.nz, L.cx, L.cy, L.cz, L.sink, L.stats);
  return hipGetLastError();
}

}  // namespace gemi
