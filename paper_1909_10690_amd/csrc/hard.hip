// Hard-binned joint histogram of fixed vs. transformed moving volume
// (Transform + Metric blocks of Fig. 1; "full histogram over all voxels",
// Discussion), for gfx950.
//
// Per call, the fixed volume is reduced to one bin byte per voxel and the
// moving volume to an "oct volume": each 16-byte element holds the clamped,
// offset intensities of a voxel's whole 2x2x2 trilinear neighbourhood as
// 16-bit values, so a lane gathers its neighbourhood with one aligned
// 128-bit load (the texture unit's 16 cycles per load, whatever its width,
// make one 16-byte gather beat two 8-byte gathers of the same bytes).
//
// One workgroup = one transform x one slab of fixed rows.  Each wave64
// walks its own run of 4-row groups with scalar coordinates; its 64 lanes
// cover a 16 x 4 tile of fixed voxels (a compact footprint in the moving
// volume even under rotation, so few cache lines per load) and step the
// exact Q32 moving coordinate by 16 * M[:,0] per iteration.  Each lane forms the exact
// 16-bit-weight x-lerps with dot products in integers (< 2^32) and the y- and
// z-lerps in fp32; the bin is read off the fp32 value, whose error is bounded
// (kBinGuard in sweep.h), unless it lies too near a bin edge: those lanes redo
// the sum in 64-bit integers, so every bin is exact.  One count goes to the
// workgroup's private joint histogram in LDS; at the end the non-zero LDS
// bins are added once into the transform's HBM histogram.
//
// 28 VALU instructions per voxel and step (37 with the y- and z-lerps in fp64
// and two instructions per x-lerp), one gather per step and one 32-bit load of
// fixed bins per four (a load of any width costs the texture unit 16 cycles a
// wave).  1000 transforms of 256x256x180 u16, 128 bins: 12.87 -> 11.99 ms a
// call.  The step now takes about 35 cycles of a CU: VALU 28, L1 accesses 26
// (64 records of 16 bytes that start anywhere), LDS 17 with conflicts.
#include "common.h"
#include "sweep.h"

#include <algorithm>
#include <mutex>
#include <utility>
#include <vector>

#pragma clang fp contract(off)

namespace gemi {

// ---------------------------------------------------------------------------
// LDS guard
// ---------------------------------------------------------------------------

namespace {
std::mutex g_lds_mu;
std::vector<std::pair<const void*, size_t>> g_lds_static;  // kernel -> static LDS bytes
size_t g_lds_device_max = 0;                               // LDS one workgroup may hold
}  // namespace

hipError_t lds_register(const void* kernel) {
  hipFuncAttributes attr;
  hipError_t e = hipFuncGetAttributes(&attr, kernel);
  if (e != hipSuccess) return e;
  int dev = 0, max_block = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&max_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev)) != hipSuccess)
    return e;
  std::lock_guard<std::mutex> g(g_lds_mu);
  g_lds_device_max = (size_t)max_block;
  for (auto& k : g_lds_static)
    if (k.first == kernel) {
      k.second = attr.sharedSizeBytes;
      return hipSuccess;
    }
  g_lds_static.emplace_back(kernel, attr.sharedSizeBytes);
  return hipSuccess;
}

hipError_t lds_guard(const void* kernel, size_t dynamic, size_t configured_max, bool at_zero) {
  for (int pass = 0; pass < 2; ++pass) {
    {
      std::lock_guard<std::mutex> g(g_lds_mu);
      for (const auto& k : g_lds_static)
        if (k.first == kernel)
          return lds_fits(dynamic, k.second, configured_max, g_lds_device_max) && (!at_zero || k.second == 0)
                     ? hipSuccess
                     : hipErrorInvalidValue;
    }
    if (pass == 0) {
      const hipError_t e = lds_register(kernel);
      if (e != hipSuccess) return e;
    }
  }
  return hipErrorInvalidValue;
}

// The arrays one after the other: each in 16-byte stores where its address
// and length allow.  Block b of nb.
__device__ __forceinline__ void clear_arrays(const ClearList& l, uint32_t b, uint32_t nb) {
  const size_t i0 = b * (size_t)256 + threadIdx.x, step = (size_t)nb * 256;
  for (int k = 0; k < l.n; ++k) {
    const size_t n = l.words[k], quads = ((uintptr_t)l.p[k] & 15) == 0 ? n / 4 : 0;
    for (size_t i = i0; i < quads; i += step) ((uint4_t*)l.p[k])[i] = uint4_t{0u, 0u, 0u, 0u};
    for (size_t i = 4 * quads + i0; i < n; i += step) l.p[k][i] = 0;
  }
}

// ---------------------------------------------------------------------------
// fixed-volume binning, once per call
// ---------------------------------------------------------------------------

// The bins in the order a hard sweep reads them (FixedOrder), four stored
// bytes of a row per thread, or in voxel order, 16 voxels per thread (a byte
// each took 111 us for 512x512x300 i16, now 46); then `used`, if
// given, gets a 1 for every bin some voxel falls in.
template <int ORDER, typename F>
__device__ __forceinline__ void prebin(int32_t nx, uint32_t rows, uint8_t* __restrict__ out,
                                       uint32_t* __restrict__ used, uint32_t block, uint32_t nb, F&& bin) {
  const uint32_t i0 = block * 256 + threadIdx.x, step = nb * 256;
  if (ORDER == kVoxelOrder) {
    __shared__ uint32_t seen[256];
    if (used) {
      seen[threadIdx.x] = 0;
      __syncthreads();
    }
    const uint32_t nvox = rows * (uint32_t)nx, n16 = nvox / 16;  // < 2^28
    for (uint32_t i = i0; i < n16; i += step) {
      uint32_t w[4] = {0, 0, 0, 0}, prev = 0x100u;
#pragma unroll
      for (uint32_t k = 0; k < 16; ++k) w[k >> 2] |= bin(16 * i + k) << (8 * (k & 3));
      if (used) {  // a run of one bin (air) marks it once
#pragma unroll
        for (uint32_t k = 0; k < 16; ++k) {
          const uint32_t b = (w[k >> 2] >> (8 * (k & 3))) & 0xFFu;
          if (b != prev && !seen[b]) seen[b] = 1u;
          prev = b;
        }
      }
      ((uint4*)out)[i] = make_uint4(w[0], w[1], w[2], w[3]);
    }
    if (block == 0 && threadIdx.x < nvox - 16 * n16) {
      const uint32_t i = 16 * n16 + threadIdx.x, b = bin(i);
      out[i] = (uint8_t)b;
      if (used) seen[b] = 1u;
    }
    if (used) {
      __syncthreads();
      if (seen[threadIdx.x]) used[threadIdx.x] = 1u;
    }
    return;
  }
  const uint32_t quads = ((uint32_t)nx + 3) / 4;
  for (uint32_t i = i0; i < rows * quads; i += step) {
    const uint32_t row = i / quads, p0 = 4 * (i - row * quads), base = row * (uint32_t)nx;
    uint32_t b[4];
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k)
      b[k] = p0 + k < (uint32_t)nx ? bin(base + (uint32_t)stored_x<ORDER>((int32_t)(p0 + k), nx)) : 0u;
    if (((base + p0) & 3) == 0 && p0 + 4 <= (uint32_t)nx) {
      *(uint32_t*)(out + base + p0) = b[0] | (b[1] << 8) | (b[2] << 16) | (b[3] << 24);
    } else {
      for (uint32_t k = 0; k < 4 && p0 + k < (uint32_t)nx; ++k) out[base + p0 + k] = (uint8_t)b[k];
    }
  }
}

// Block `block` of nb of the binning of volume f into `bins` bins; div: of its
// integer range.
template <int ORDER>
__device__ __forceinline__ void prebin_volume(const VolumeDesc& f, int32_t bins, Divider div, uint8_t* __restrict__ out,
                                              uint32_t* __restrict__ used, uint32_t block, uint32_t nb) {
  const uint32_t rows = (uint32_t)f.ny * (uint32_t)f.nz;
  const int32_t lo = (int32_t)f.lo, hi = (int32_t)f.hi;
  auto whole = [&]<typename T>(const T* __restrict__ u) {
    prebin<ORDER>(f.nx, rows, out, used, block, nb,
                  [&](uint32_t i) { return fixed_bin_int((int32_t)u[i], lo, hi, (uint32_t)bins, div); });
  };
  switch (f.dtype) {  // the same for every thread
  case 0: whole((const uint8_t*)f.data); break;
  case 1: whole((const uint16_t*)f.data); break;
  case 2: whole((const int16_t*)f.data); break;
  default: {
    const float* __restrict__ u = (const float*)f.data;
    prebin<ORDER>(f.nx, rows, out, used, block, nb,
                  [&](uint32_t i) { return fixed_bin_real((double)u[i], f.lo, f.hi, bins); });
  }
  }
}

static Divider fixed_divider(const VolumeDesc& f) {
  return f.dtype == 3 ? Divider{0, 0} : make_divider((uint32_t)((int32_t)f.hi - (int32_t)f.lo + 1));
}

__global__ __launch_bounds__(256) void prebin_kernel(VolumeDesc f, int32_t bins, Divider div,
                                                     uint8_t* __restrict__ out, uint32_t* __restrict__ used) {
  prebin_volume<kVoxelOrder>(f, bins, div, out, used, blockIdx.x, gridDim.x);
}

hipError_t launch_prebin_voxels(const VolumeDesc& f, int bins, uint8_t* out, uint32_t* used, hipStream_t s) {
  const size_t nvox = (size_t)f.nx * f.ny * f.nz;
  hipLaunchKernelGGL(prebin_kernel, dim3(fill_blocks(nvox / 16)), dim3(256), 0, s, f, bins, fixed_divider(f), out, used);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// moving oct volume, once per call
// ---------------------------------------------------------------------------

// A preparation block's row part: 256 voxels of row (y, z).
struct RowBlock {
  int32_t x0, y, z;
  __device__ __forceinline__ RowBlock(int32_t nx, int32_t ny, uint32_t block) {
    const uint32_t per = ((uint32_t)nx + 255) / 256, row = block / per;
    x0 = (int32_t)(256 * (block - row * per));
    z = (int32_t)(row / (uint32_t)ny);
    y = (int32_t)(row - (uint32_t)z * (uint32_t)ny);
  }
};

// out[z][y][x] holds the eight 16-bit clamped, offset intensities
// v' = clamp(v, lo, hi) - lo of the voxel's 2x2x2 neighbourhood, so one
// 16-byte load fetches all trilinear corners: word 2 dz + dy packs
// (x, y+dy, z+dz) in its low half and (x1, y+dy, z+dz) in its high half,
// with x1 = min(x+1, nx-1) and y+1, z+1 likewise clamped.  A neighbour
// index is thus clamped to the volume, as in the trilinear rule; on those
// corners the hard path's weight is 0, and the Parzen path's derivative
// along that axis vanishes.
// DIFF (kOctD): each word holds -(v0' + v1') in its low half and v1' - v0' in
// its high half instead.
// Block `block`: 256 voxels of a row.
template <typename T, bool DIFF>
__device__ __forceinline__ void pack_octs(const T* __restrict__ v, int32_t nx, int32_t ny, int32_t nz, int32_t lo,
                                          int32_t hi, uint4* __restrict__ out, uint32_t block) {
  const RowBlock rb(nx, ny, block);
  const int32_t y = rb.y, z = rb.z;
  uint4* __restrict__ orow = out + ((size_t)z * ny + y) * nx;
  const T* __restrict__ r00 = v + ((size_t)z * ny + y) * nx;
  const T* __restrict__ r10 = r00 + (y + 1 < ny ? nx : 0);
  const size_t dz = z + 1 < nz ? (size_t)nx * ny : 0;
  const T* __restrict__ r01 = r00 + dz;
  const T* __restrict__ r11 = r10 + dz;
  auto c = [&](T raw) -> uint32_t { return clamp_offset((int32_t)raw, lo, hi); };
  const int32_t x = rb.x0 + (int32_t)threadIdx.x;
  if (x < nx) {
    const int32_t x1 = x + 1 < nx ? x + 1 : nx - 1;
    auto pair = [&](const T* r) -> uint32_t {
      const uint32_t v0 = c(r[x]), v1 = c(r[x1]);
      return DIFF ? ((0u - v0 - v1) & 0xFFFFu) | ((v1 - v0) << 16) : v0 | (v1 << 16);
    };
    orow[x] = make_uint4(pair(r00), pair(r10), pair(r01), pair(r11));
  }
}

// The same neighbourhood with 8-bit corners (moving range R <= 256): byte
// 4 dz + 2 dy + dx' of the element holds (x + dx', y + dy, z + dz), dx' = 0
// for x and 1 for x1.
template <typename T>
__device__ __forceinline__ void pack_oct8(const T* __restrict__ v, int32_t nx, int32_t ny, int32_t nz, int32_t lo,
                                          int32_t hi, uint2* __restrict__ out, uint32_t block) {
  const RowBlock rb(nx, ny, block);
  const int32_t y = rb.y, z = rb.z;
  uint2* __restrict__ orow = out + ((size_t)z * ny + y) * nx;
  const T* __restrict__ r00 = v + ((size_t)z * ny + y) * nx;
  const T* __restrict__ r10 = r00 + (y + 1 < ny ? nx : 0);
  const size_t dz = z + 1 < nz ? (size_t)nx * ny : 0;
  const T* __restrict__ r01 = r00 + dz;
  const T* __restrict__ r11 = r10 + dz;
  auto c = [&](T raw) -> uint32_t { return clamp_offset((int32_t)raw, lo, hi); };
  const int32_t x = rb.x0 + (int32_t)threadIdx.x;
  if (x < nx) {
    const int32_t x1 = x + 1 < nx ? x + 1 : nx - 1;
    orow[x] = make_uint2(c(r00[x]) | (c(r00[x1]) << 8) | (c(r10[x]) << 16) | (c(r10[x1]) << 24),
                         c(r01[x]) | (c(r01[x1]) << 8) | (c(r11[x]) << 16) | (c(r11[x1]) << 24));
  }
}

// Octs in tiles (tiled_index), one record per thread: records of a tile are
// neighbours in memory, so the stores are whole lines and the reads of a
// tile's eight or sixteen records mostly hit the same ones (256x256x180 u16:
// 88 us against 36 for rows of octs, see hard_gather).
template <typename T, int BASE>
__device__ __forceinline__ void pack_tiled(const T* __restrict__ v, int32_t nx, int32_t ny, int32_t nz, int32_t lo,
                                           int32_t hi, void* __restrict__ out, uint32_t block, uint32_t nb) {
  constexpr uint32_t kx = BASE == kOct8 ? 4 : 2;  // tile width
  const uint32_t px = (uint32_t)tile_pad_x(nx, BASE == kOct8), py = (uint32_t)tile_pad(ny);
  const uint32_t n = (uint32_t)tiled_records(nx, ny, nz, BASE == kOct8);  // < 2^29
  auto c = [&](uint32_t i) -> uint32_t { return clamp_offset((int32_t)v[i], lo, hi); };
  for (uint32_t i = block * 256 + threadIdx.x; i < n; i += nb * 256) {
    const uint32_t tile = i / (4 * kx), low = i - tile * (4 * kx);
    const uint32_t tr = tile / (px / kx), tz = tr / (py / 2);
    const uint32_t x = (tile - tr * (px / kx)) * kx + low % kx;
    const uint32_t y = (tr - tz * (py / 2)) * 2 + low / kx % 2, z = 2 * tz + low / (2 * kx);
    if (x >= (uint32_t)nx || y >= (uint32_t)ny || z >= (uint32_t)nz) continue;  // padding: never gathered
    const uint32_t a = (z * (uint32_t)ny + y) * (uint32_t)nx + x;
    const uint32_t dx = x + 1 < (uint32_t)nx ? 1 : 0, dy = y + 1 < (uint32_t)ny ? (uint32_t)nx : 0;
    const uint32_t dz = z + 1 < (uint32_t)nz ? (uint32_t)nx * (uint32_t)ny : 0;
    if (BASE == kOct8) {
      ((uint2*)out)[i] = make_uint2(c(a) | (c(a + dx) << 8) | (c(a + dy) << 16) | (c(a + dy + dx) << 24),
                                    c(a + dz) | (c(a + dz + dx) << 8) | (c(a + dz + dy) << 16) | (c(a + dz + dy + dx) << 24));
    } else {
      auto pair = [&](uint32_t r) -> uint32_t {
        const uint32_t v0 = c(r), v1 = c(r + dx);
        return BASE == kOctD ? ((0u - v0 - v1) & 0xFFFFu) | ((v1 - v0) << 16) : v0 | (v1 << 16);
      };
      ((uint4*)out)[i] = make_uint4(pair(a), pair(a + dy), pair(a + dz), pair(a + dz + dy));
    }
  }
}

// out[i] = clamp(v[i], lo, hi) - lo as 16 bits (moving_copy_bytes), 8 voxels
// per lane with one load and one 16-byte store where the source is aligned
// to 8 voxels.
template <typename T>
__device__ __forceinline__ void pack_copy(const T* __restrict__ v, size_t nvox, int32_t lo, int32_t hi,
                                          uint16_t* __restrict__ out, uint32_t block, uint32_t nb) {
  typedef const __attribute__((address_space(1))) T gT;
  const size_t i0 = block * (size_t)256 + threadIdx.x, step = (size_t)nb * 256;
  const size_t n8 = ((uintptr_t)v & (8 * sizeof(T) - 1)) == 0 ? nvox / 8 : 0;
  for (size_t i = i0; i < n8; i += step) ((vec4u*)out)[i] = load_offset8((gT*)v + 8 * i, lo, hi);
  for (size_t i = 8 * n8 + i0; i < nvox; i += step) out[i] = (uint16_t)clamp_offset((int32_t)v[i], lo, hi);
}

// Block `block` of nb of an integer moving volume in layout `gather`.
__device__ __forceinline__ void pack_volume(const VolumeDesc& m, int32_t gather, void* __restrict__ out, uint32_t block,
                                            uint32_t nb) {
  const int32_t lo = (int32_t)m.lo, hi = (int32_t)m.hi;
  const uint32_t parts = row_parts(m.nx, m.ny, m.nz);
  auto whole = [&]<typename T>(const T* __restrict__ v) {
    switch (gather) {
    case kOct16:
      for (uint32_t b = block; b < parts; b += nb) pack_octs<T, false>(v, m.nx, m.ny, m.nz, lo, hi, (uint4*)out, b);
      break;
    case kOctD:
      for (uint32_t b = block; b < parts; b += nb) pack_octs<T, true>(v, m.nx, m.ny, m.nz, lo, hi, (uint4*)out, b);
      break;
    case kOct8:
      for (uint32_t b = block; b < parts; b += nb) pack_oct8(v, m.nx, m.ny, m.nz, lo, hi, (uint2*)out, b);
      break;
    case kCopy16: pack_copy(v, (size_t)m.nx * m.ny * m.nz, lo, hi, (uint16_t*)out, block, nb); break;
    case kOct16 | kTiled: pack_tiled<T, kOct16>(v, m.nx, m.ny, m.nz, lo, hi, out, block, nb); break;
    case kOctD | kTiled: pack_tiled<T, kOctD>(v, m.nx, m.ny, m.nz, lo, hi, out, block, nb); break;
    case kOct8 | kTiled: pack_tiled<T, kOct8>(v, m.nx, m.ny, m.nz, lo, hi, out, block, nb); break;
    }
  };
  switch (m.dtype) {  // the same for every thread
  case 0: whole((const uint8_t*)m.data); break;
  case 1: whole((const uint16_t*)m.data); break;
  case 2: whole((const int16_t*)m.data); break;
  }
}

static unsigned pack_blocks(const VolumeDesc& m, int32_t gather) {
  const size_t nvox = (size_t)m.nx * m.ny * m.nz;
  // (each block waits for the matrices first: as many as the chip holds at once,
  // 256x256x180 u16 20.8 us a launch, in 5760 blocks 24.4)
  if (gather & kChoose) return std::min(fill_blocks((nvox + 7) / 8), 2048u);
  if (gather == kCopy16) return fill_blocks((nvox + 7) / 8);
  if (gather & kTiled) return fill_blocks(tiled_records(m.nx, m.ny, m.nz, gather_base(gather) == kOct8));
  return row_part_blocks(row_parts(m.nx, m.ny, m.nz));
}

// ---------------------------------------------------------------------------
// what a call does before its sweep
// ---------------------------------------------------------------------------

struct PrepareArgs {
  Prepare p;
  Divider div;
  PrepareBlocks blocks;
};

// Whether a few transforms take octs (octs_weight), by 4 x 4 x 4 points of the
// fixed volume, a lane each: the same in every wave.  A lane loads an entry of
// the matrices (n <= 4), so that the waves wait once: each packs few voxels.
__device__ __forceinline__ bool turned_octs(const Prepare& p) {
  static_assert(12 * kCopyTransforms <= 64, "an entry a lane");
  const int lane = threadIdx.x & 63;
  const float entry = lane < 12 * (int)p.n ? (float)p.P[lane] : 0.0f;
  const Geometry& g = p.geo;
  const float x = (float)g.forg[0] + (float)g.fsp[0] * (((float)(lane & 3) + 0.5f) * 0.25f * (float)(p.f.nx - 1));
  const float y = (float)g.forg[1] + (float)g.fsp[1] * (((float)((lane >> 2) & 3) + 0.5f) * 0.25f * (float)(p.f.ny - 1));
  const float z = (float)g.forg[2] + (float)g.fsp[2] * (((float)(lane >> 4) + 0.5f) * 0.25f * (float)(p.f.nz - 1));
  const float size[3] = {(float)g.msp[0] * (float)(p.m.nx - 1), (float)g.msp[1] * (float)(p.m.ny - 1),
                         (float)g.msp[2] * (float)(p.m.nz - 1)};
  const float rise_y = 0.5f * (float)g.fsp[0] / (float)g.msp[1], rise_z = (float)g.fsp[0] / (float)g.msp[2];
  float sum = 0.0f;
  for (int t = 0; t < (int)p.n; ++t) {
    auto P = [&](int e) {
      return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, entry), 12 * t + e));
    };
    bool in = true;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const float q = P(4 * r) * x + P(4 * r + 1) * y + P(4 * r + 2) * z + P(4 * r + 3) - (float)g.morg[r];
      in = in && q >= 0.0f && q <= size[r];
    }
    const float inside = p.clamp ? 64.0f : (float)__popcll(__builtin_amdgcn_ballot_w64(in));
    const float rho = fminf(fabsf(P(4)) * rise_y + fabsf(P(8)) * rise_z, 1.0f);  // 1 for a NaN
    sum += inside * (0.3f + 1.7f * rho * rho);
  }
  return sum * p.weight > 64.0f;
}

// The parts depend on nothing but the caller's inputs, so they share a launch,
// the longest first: a small call (48^3, one transform) is mostly launches of
// 2 to 3 us.
__global__ __launch_bounds__(256, 8) void prepare_kernel(PrepareArgs a) {
  uint32_t block = blockIdx.x;
  const PrepareBlocks& nb = a.blocks;
  if (block < nb.pack) {
    int32_t gather = a.p.records && *a.p.records ? (int32_t)kOct16 : a.p.gather;
    if (gather & kChoose) {
      gather = a.p.weight > 0.0f && turned_octs(a.p) ? gather & ~kChoose : (int32_t)kCopy16;
      if (a.p.choice && block == 0 && threadIdx.x == 0) a.p.choice[0] = gather == kCopy16 ? 0u : 1u;
    }
    pack_volume(a.p.m, gather, a.p.gvol, block, nb.pack);
    return;
  }
  block -= nb.pack;
  if (block < nb.bin) {
    switch (a.p.order) {
    case kRunOrder: prebin_volume<kRunOrder>(a.p.f, a.p.bins, a.div, a.p.fbins, nullptr, block, nb.bin); break;
    case kCubeOrder: prebin_volume<kCubeOrder>(a.p.f, a.p.bins, a.div, a.p.fbins, nullptr, block, nb.bin); break;
    default: prebin_volume<kVoxelOrder>(a.p.f, a.p.bins, a.div, a.p.fbins, nullptr, block, nb.bin);
    }
    return;
  }
  block -= nb.bin;
  if (block < nb.clear) {
    clear_arrays(a.p.clear, block, nb.clear);
    return;
  }
  block -= nb.clear;
  if (a.p.choice && block == 0 && threadIdx.x < 64) {  // n <= kCopyTransforms
    const float per = (float)a.p.geo.fsp[0] / (float)a.p.geo.msp[2];
    float rise = (int64_t)threadIdx.x < a.p.n ? fminf(fabsf((float)a.p.P[12 * threadIdx.x + 8]) * per, 1.0f) : 0.0f;
    for (int off = 32; off > 0; off >>= 1) rise += __shfl_xor(rise, off, 64);
    if (threadIdx.x == 0) a.p.choice[1] = rise > kTurnedRise * (float)a.p.n ? 1u : 0u;
  }
  for (int64_t t = block * 256ll + threadIdx.x; t < a.p.n; t += nb.compose * 256ll) {
    double m[12];
    compose_index_matrix(a.p.P + 12 * t, a.p.geo, m);
#pragma unroll
    for (int e = 0; e < 12; ++e) a.p.M[12 * t + e] = m[e];
  }
}

hipError_t launch_prepare(const Prepare& p, hipStream_t s) {
  PrepareArgs a{p, Divider{0, 0}, {}};
  PrepareBlocks& nb = a.blocks;
  if (p.gvol) {
    if (p.m.dtype > 2) return hipErrorInvalidValue;
    if (p.weight > 0.0f && (!p.choice || !p.P || !p.fbins)) return hipErrorInvalidValue;
    nb.pack = pack_blocks(p.m, p.gather);
  }
  if (p.fbins) {
    a.div = fixed_divider(p.f);
    const size_t rows = (size_t)p.f.ny * p.f.nz;
    nb.bin = fill_blocks(p.order == kVoxelOrder ? rows * p.f.nx / 16 : rows * ((p.f.nx + 3) / 4));
  }
  size_t most = 0;
  for (int k = 0; k < p.clear.n; ++k) most = p.clear.words[k] > most ? p.clear.words[k] : most;
  if (most) nb.clear = fill_blocks((most + 3) / 4);
  if (p.P && p.n > 0) nb.compose = std::min(fill_blocks((size_t)p.n), 4096u);
  if (p.choice && p.n > kCopyTransforms) return hipErrorInvalidValue;
  if (nb.total() == 0) return hipSuccess;
  if (!nb.fits()) return hipErrorInvalidValue;
  hipLaunchKernelGGL(prepare_kernel, dim3(nb.total()), dim3(256), 0, s, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// the histogram sweep
// ---------------------------------------------------------------------------

// Dynamic LDS limit of the hard sweeps (a u32 table up to 128 bins, 16-bit
// pairs above: at most 128 KiB), within the 160 KiB of a workgroup.
constexpr size_t kHardLdsMax = 160 * 1024;

struct HardArgs {
  const double* transforms;
  uint32_t* hist;
  uint64_t* count;
  HardGeom geom;
  SlabSplit split[2];       // [1] where choice[1] is not 0
  const uint32_t* choice;   // Prepare::choice, or NULL
  int32_t n;
  int32_t slab_major;     // 1: consecutive workgroups of an XCD share a slab
  int32_t deal;           // bricks: slabs in turn over the XCDs (deal_slabs)
  const uint32_t* order;  // processing order (absolute indices) or NULL
  uint32_t order_base;    // absolute index of this launch's first transform
};

// 1024-thread workgroups are held to 64 VGPRs (a few row-loop values spill to
// scratch) so that two of them, 8 waves per SIMD, share a CU next to two
// 64 KiB LDS histograms; the sweep waits on its gathers and gains from the
// extra waves.  Smaller workgroups keep their registers.
// BRICK: slabs as bricks (sweep_rods) rather than thin slabs.
template <bool CLAMP, bool PACKED, int GL, int NT, bool BRICK = false>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == 1024 ? 8 : 1)))
void hist_hard_kernel(HardArgs a) {
  extern __shared__ uint32_t lds_hist[];
  const int B = a.geom.bins;
  SlabSplit split = a.split[0];
  bool octs = false;
  if constexpr (!BRICK) {
    if (a.choice) {
      octs = (GL & kChoose) != 0 && a.choice[0] != 0;
      if (a.choice[1]) split = a.split[1];
      // the launch is made for the larger count
      if ((blockIdx.x >> 3) >= (uint32_t)(split.chunks >> 3) * (uint32_t)a.n) return;
    }
  }
  clear_hist<PACKED, NT>(lds_hist, B);
  uint32_t t, chunk, band;
  block_work(split.chunks, a.n, 1, a.slab_major, t, chunk, band);
  if (BRICK && a.deal) chunk = dealt_slab(chunk, (uint32_t)split.chunks);
  if (a.order) t = a.order[t] - a.order_base;
  const double* Md = a.transforms + 12 * (size_t)t;
  int64_t Mq[12];
  const bool ok = quantize_transform_wave(Md, Mq);
  __syncthreads();
  if (ok) {
    if constexpr (BRICK) {
      sweep_rods<CLAMP, PACKED, GL, NT / 64>(a.geom, Md, Mq, split.chunks, chunk, lds_hist);
    } else if constexpr ((GL & kChoose) != 0) {
      if (octs)
        sweep_hard<CLAMP, PACKED, GL & ~kChoose, NT / 64>(a.geom, Md, Mq, split, chunk, lds_hist);
      else
        sweep_hard<CLAMP, PACKED, kCopy16, NT / 64>(a.geom, Md, Mq, split, chunk, lds_hist);
    } else {
      sweep_hard<CLAMP, PACKED, GL, NT / 64>(a.geom, Md, Mq, split, chunk, lds_hist);
    }
  }
  __syncthreads();
  if (ok) flush_hist<PACKED, NT>(lds_hist, B, a.hist + (size_t)t * B * B, a.count + t, false);
}

// Sampled sweep: the workgroup's share of the sample list (entries
// {x | y << 12 | fixed bin << 24, z}) for one transform, each sample's Q32
// coordinates formed straight from the matrix.  With 16-bit counters the
// share is counted in spans of at most 65535 samples, each flushed before
// the next, so no counter can overflow whatever the sample count.
template <bool CLAMP, bool PACKED, int GL, int NT>
__global__ __launch_bounds__(NT) void hist_sampled_kernel(HardArgs a, const uint2* __restrict__ list,
                                                          const unsigned long long* __restrict__ n_list) {
  extern __shared__ uint32_t lds_hist[];
  const int B = a.geom.bins;
  clear_hist<PACKED, NT>(lds_hist, B);
  uint32_t t, chunk, band;
  const int32_t chunks = a.split[0].chunks;
  block_work(chunks, a.n, 1, a.slab_major, t, chunk, band);
  int64_t Mq[12];
  const bool ok = quantize_transform(a.transforms + 12 * (size_t)t, Mq);
  const int64_t ns = (int64_t)*n_list;
  const int64_t s0 = ns * chunk / chunks, s1 = ns * (chunk + 1) / chunks;
  const int64_t span = PACKED ? 65535 : s1 - s0;
  const HardStep hs(a.geom, PACKED, GL);
  uint32_t* out = a.hist + (size_t)t * B * B;
  for (int64_t p0 = s0; p0 < s1; p0 += span) {
    const int64_t p1 = p0 + span < s1 ? p0 + span : s1;
    __syncthreads();
    if (ok) {
      for (int64_t e = p0 + threadIdx.x; e < p1; e += NT) {
        const uint2 en = list[e];
        const int64_t x = en.x & 0xFFFu, y = (en.x >> 12) & 0xFFFu, z = en.y;
        const uint32_t fb = en.x >> 24;
        const int64_t qx = Mq[0] * x + Mq[1] * y + Mq[2] * z + Mq[3];
        const int64_t qy = Mq[4] * x + Mq[5] * y + Mq[6] * z + Mq[7];
        const int64_t qz = Mq[8] * x + Mq[9] * y + Mq[10] * z + Mq[11];
        hs.count<CLAMP, PACKED, GL>(qx, qy, qz, [&] { return fb; }, lds_hist);
      }
    }
    __syncthreads();
    if (ok) flush_hist<PACKED, NT>(lds_hist, B, out, a.count + t, true);
  }
}

// Threads per workgroup of a sampled sweep: 512, or 1024 where the table
// leaves room for fewer than four workgroups in a CU's 160 KiB of LDS (above
// about 100 bins): the sweep waits on its gathers and needs the waves (256
// bins, 25% of 181x217x181, 150 affines: 2.34 -> 1.95 ms a call).
static int32_t sampled_block(size_t lds) { return 4 * lds > 160 * 1024 ? 1024 : 512; }

template <bool CLAMP, bool PACKED, int GL, int NT>
static hipError_t launch_sampled_nt(const HardArgs& a, const uint2* list, const unsigned long long* n_list,
                                    size_t lds, hipStream_t s) {
  const hipError_t e = lds_guard((const void*)hist_sampled_kernel<CLAMP, PACKED, GL, NT>, lds, kHardLdsMax, true);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((hist_sampled_kernel<CLAMP, PACKED, GL, NT>), dim3((unsigned)(a.n * a.split[0].chunks)), dim3(NT),
                     lds, s, a, list, n_list);
  return hipGetLastError();
}

template <bool CLAMP, bool PACKED, int GL>
static hipError_t launch_sampled_variant(const HardArgs& a, const uint2* list, const unsigned long long* n_list,
                                         size_t lds, hipStream_t s) {
  return sampled_block(lds) == 1024 ? launch_sampled_nt<CLAMP, PACKED, GL, 1024>(a, list, n_list, lds, s)
                                    : launch_sampled_nt<CLAMP, PACKED, GL, 512>(a, list, n_list, lds, s);
}

template <bool CLAMP, bool PACKED, int GL, int NT, bool BRICK>
static hipError_t launch_variant(const HardArgs& a, int n, size_t lds, hipStream_t s) {
  const hipError_t e =
      lds_guard((const void*)hist_hard_kernel<CLAMP, PACKED, GL, NT, BRICK>, lds, kHardLdsMax, true);
  if (e != hipSuccess) return e;
  const int32_t chunks = a.choice ? std::max(a.split[0].chunks, a.split[1].chunks) : a.split[0].chunks;
  hipLaunchKernelGGL((hist_hard_kernel<CLAMP, PACKED, GL, NT, BRICK>), dim3((unsigned)(n * chunks)), dim3(NT), lds, s, a);
  return hipGetLastError();
}

template <int GL, int NT, bool BRICK>
static hipError_t launch_layout(const HardArgs& a, int n, bool clamp, bool packed, size_t lds,
                                hipStream_t s) {
  if (clamp)
    return packed ? launch_variant<true, true, GL, NT, BRICK>(a, n, lds, s)
                  : launch_variant<true, false, GL, NT, BRICK>(a, n, lds, s);
  return packed ? launch_variant<false, true, GL, NT, BRICK>(a, n, lds, s)
                : launch_variant<false, false, GL, NT, BRICK>(a, n, lds, s);
}

template <int NT, bool BRICK = false>
static hipError_t launch_nt(const HardArgs& a, int n, bool clamp, bool packed, size_t lds,
                            hipStream_t s) {
  switch (a.geom.gather) {
  case kOct8: return launch_layout<kOct8, NT, BRICK>(a, n, clamp, packed, lds, s);
  case kOctD: return launch_layout<kOctD, NT, BRICK>(a, n, clamp, packed, lds, s);
  case kOct16: return launch_layout<kOct16, NT, BRICK>(a, n, clamp, packed, lds, s);
  }
  if constexpr (BRICK) {  // tiles serve bricks only, the copy few transforms in thin slabs
    switch (a.geom.gather) {
    case kOct8 | kTiled: return launch_layout<kOct8 | kTiled, NT, BRICK>(a, n, clamp, packed, lds, s);
    case kOctD | kTiled: return launch_layout<kOctD | kTiled, NT, BRICK>(a, n, clamp, packed, lds, s);
    case kOct16 | kTiled: return launch_layout<kOct16 | kTiled, NT, BRICK>(a, n, clamp, packed, lds, s);
    default: return hipErrorInvalidValue;
    }
  } else {
    switch (a.geom.gather) {
    case kCopy16: return launch_layout<kCopy16, NT, BRICK>(a, n, clamp, packed, lds, s);
    case kOct8 | kChoose: return launch_layout<kOct8 | kChoose, NT, BRICK>(a, n, clamp, packed, lds, s);
    case kOctD | kChoose: return launch_layout<kOctD | kChoose, NT, BRICK>(a, n, clamp, packed, lds, s);
    case kOct16 | kChoose: return launch_layout<kOct16 | kChoose, NT, BRICK>(a, n, clamp, packed, lds, s);
    default: return hipErrorInvalidValue;
    }
  }
}

HardGeom make_hard_geom(const VolumeDesc& fixed, const VolumeDesc& moving, const uint8_t* fbins,
                        const void* gvol, int32_t gather, int32_t bins) {
  HardGeom g;
  g.fbins = fbins;
  g.gvol = gvol;
  g.gather = gather;
  g.fnx = fixed.nx;
  g.fny = fixed.ny;
  g.fnz = fixed.nz;
  g.mnx = moving.nx;
  g.mny = moving.ny;
  g.mnz = moving.nz;
  g.gvol_bytes = (uint32_t)gather_volume_bytes(gather, moving.nx, moving.ny, moving.nz);
  g.bins = bins;
  g.rods = rods_for(fixed.nx, fixed.ny, fixed.nz);
  const uint32_t R = (uint32_t)((int32_t)moving.hi - (int32_t)moving.lo + 1);
  g.scale = ldexp((double)bins / (double)R, -48);
  g.div = make_divider(R);
  return g;
}

hipError_t launch_hist_hard(const HardLaunch& L, hipStream_t s) {
  if (L.n == 0) return hipSuccess;
  HardArgs a;
  a.transforms = L.transforms;
  a.hist = L.hist;
  a.count = L.count;
  a.geom = make_hard_geom(L.fixed, L.moving, L.fbins, L.gvol, L.gather, L.bins);
  a.split[0] = L.split[0];
  a.split[1] = L.split[1];
  a.choice = L.choice;
  a.n = L.n;
  a.slab_major = L.slab_major;
  a.deal = deal_slabs(L.fixed.nx, L.fixed.ny, L.fixed.nz) ? 1 : 0;
  a.order = nullptr;
  a.order_base = 0;
  const size_t lds = hist_lds_bytes(L.bins, L.packed);
  if (L.block != 256 && L.block != 512 && L.block != 1024) return hipErrorInvalidValue;
  int32_t step = transforms_per_launch(std::max(L.split[0].chunks, L.split[1].chunks), L.block);
  // with an order, launches start at multiples of its sorted blocks
  const bool ordered = L.order && step >= kOrderBlock;
  if (ordered) step -= step % kOrderBlock;
  for (int32_t t0 = 0; t0 < L.n; t0 += step) {
    HardArgs b = a;
    b.n = L.n - t0 < step ? L.n - t0 : step;
    b.transforms = a.transforms + 12 * (size_t)t0;
    b.hist = a.hist + (size_t)t0 * L.bins * L.bins;
    b.count = a.count + t0;
    if (ordered) {
      b.order = L.order + t0;
      b.order_base = (uint32_t)(L.order_t0 + t0);
    }
    hipError_t e;
    switch (L.block) {
    case 256: e = launch_nt<256>(b, b.n, L.clamp, L.packed, lds, s); break;
    case 512: e = launch_nt<512>(b, b.n, L.clamp, L.packed, lds, s); break;
    default:  // 1024; bricks only with the default 1024-thread shape
      e = L.brick ? launch_nt<1024, true>(b, b.n, L.clamp, L.packed, lds, s)
                  : launch_nt<1024>(b, b.n, L.clamp, L.packed, lds, s);
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_hist_sampled(const HardLaunch& L, const uint2* list, const unsigned long long* n_list,
                               hipStream_t s) {
  if (L.n == 0) return hipSuccess;
  HardArgs a;
  a.transforms = L.transforms;
  a.hist = L.hist;
  a.count = L.count;
  a.geom = make_hard_geom(L.fixed, L.moving, L.fbins, L.gvol, L.gather, L.bins);
  a.split[0] = a.split[1] = L.split[0];
  a.choice = nullptr;
  a.n = L.n;
  a.slab_major = 1;
  a.deal = 0;
  a.order = nullptr;  // the sampled sweep keeps the batch order
  a.order_base = 0;
  const size_t lds = hist_lds_bytes(L.bins, L.packed);
  auto layout = [&]<int GL>(const HardArgs& b) -> hipError_t {
    if (L.clamp)
      return L.packed ? launch_sampled_variant<true, true, GL>(b, list, n_list, lds, s)
                      : launch_sampled_variant<true, false, GL>(b, list, n_list, lds, s);
    return L.packed ? launch_sampled_variant<false, true, GL>(b, list, n_list, lds, s)
                    : launch_sampled_variant<false, false, GL>(b, list, n_list, lds, s);
  };
  auto one = [&](const HardArgs& b) -> hipError_t {
    switch (b.geom.gather) {
    case kOct8: return layout.template operator()<kOct8>(b);
    case kOctD: return layout.template operator()<kOctD>(b);
    case kOct16: return layout.template operator()<kOct16>(b);
    default: return hipErrorInvalidValue;
    }
  };
  const int32_t step = transforms_per_launch(L.split[0].chunks, sampled_block(lds));
  for (int32_t t0 = 0; t0 < L.n; t0 += step) {
    HardArgs b = a;
    b.n = L.n - t0 < step ? L.n - t0 : step;
    b.transforms = a.transforms + 12 * (size_t)t0;
    b.hist = a.hist + (size_t)t0 * L.bins * L.bins;
    b.count = a.count + t0;
    const hipError_t e = one(b);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int GL, int NT, bool BRICK = false>
static hipError_t allow_big_lds() {
  const int bytes = (int)kHardLdsMax;
  const void* fns[4] = {(const void*)hist_hard_kernel<false, false, GL, NT, BRICK>,
                        (const void*)hist_hard_kernel<true, false, GL, NT, BRICK>,
                        (const void*)hist_hard_kernel<false, true, GL, NT, BRICK>,
                        (const void*)hist_hard_kernel<true, true, GL, NT, BRICK>};
  for (const void* f : fns) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess || (e = lds_register(f)) != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int NT>
static hipError_t allow_big_lds_nt() {
  hipError_t e;
  if ((e = allow_big_lds<kOct16, NT>()) != hipSuccess) return e;
  if ((e = allow_big_lds<kOct8, NT>()) != hipSuccess) return e;
  if ((e = allow_big_lds<kOctD, NT>()) != hipSuccess) return e;
  if ((e = allow_big_lds<kOct16 | kChoose, NT>()) != hipSuccess) return e;
  if ((e = allow_big_lds<kOct8 | kChoose, NT>()) != hipSuccess) return e;
  if ((e = allow_big_lds<kOctD | kChoose, NT>()) != hipSuccess) return e;
  return allow_big_lds<kCopy16, NT>();
}

template <int GL, int NT>
static hipError_t allow_sampled_lds() {
  const void* fns[4] = {(const void*)hist_sampled_kernel<false, false, GL, NT>,
                        (const void*)hist_sampled_kernel<true, false, GL, NT>,
                        (const void*)hist_sampled_kernel<false, true, GL, NT>,
                        (const void*)hist_sampled_kernel<true, true, GL, NT>};
  for (const void* f : fns) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kHardLdsMax);
    if (e != hipSuccess || (e = lds_register(f)) != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int NT>
static hipError_t allow_sampled_lds_nt() {
  hipError_t e;
  if ((e = allow_sampled_lds<kOct16, NT>()) != hipSuccess) return e;
  if ((e = allow_sampled_lds<kOct8, NT>()) != hipSuccess) return e;
  return allow_sampled_lds<kOctD, NT>();
}

hipError_t configure_hard_kernels() {
  hipError_t e;
  if ((e = allow_sampled_lds_nt<512>()) != hipSuccess) return e;
  if ((e = allow_sampled_lds_nt<1024>()) != hipSuccess) return e;
  if ((e = allow_big_lds_nt<256>()) != hipSuccess) return e;
  if ((e = allow_big_lds_nt<512>()) != hipSuccess) return e;
  if ((e = allow_big_lds_nt<1024>()) != hipSuccess) return e;
  if ((e = allow_big_lds<kOct16, 1024, true>()) != hipSuccess) return e;
  if ((e = allow_big_lds<kOctD, 1024, true>()) != hipSuccess) return e;
  if ((e = allow_big_lds<kOct8, 1024, true>()) != hipSuccess) return e;
  if ((e = allow_big_lds<kOct16 | kTiled, 1024, true>()) != hipSuccess) return e;
  if ((e = allow_big_lds<kOctD | kTiled, 1024, true>()) != hipSuccess) return e;
  return allow_big_lds<kOct8 | kTiled, 1024, true>();
}

// ---------------------------------------------------------------------------
// processing order of a batch
// ---------------------------------------------------------------------------

// A thin slab of the fixed volume spans every x and y, so its image in the
// moving volume is set by the moving z that each transform assigns to it:
// workgroups that sweep one slab for transforms of similar z rows read the
// same moving slices, which then stay in the XCD's L2.  Transforms are
// keyed by four features of the index-space z row (M[2][.]) in moving
// voxels: the image depth of the fixed centre, and how much that depth
// changes across the fixed volume's z, x and y extents; the quantised
// features are interleaved bit by bit (a Morton code), with the index in
// the low bits, and each block of kOrderBlock transforms is sorted by that
// key (bitonic, in LDS).  The histograms do not depend on the order.
__global__ __launch_bounds__(1024) void order_transforms_kernel(const double* __restrict__ M, int32_t n,
                                                                float cx, float cy, float cz, float ex, float ey,
                                                                float ez, uint32_t* __restrict__ order) {
  __shared__ unsigned long long key[kOrderBlock];
  const int32_t base = (int32_t)blockIdx.x * kOrderBlock;
  const int32_t m = min(kOrderBlock, n - base);
  int32_t p = 1;
  while (p < m) p <<= 1;
  auto quant = [](float f) -> uint32_t {  // 13 bits, 2 moving voxels per step
    const float v = floorf(f * 0.5f) + 4096.0f;
    return (uint32_t)fminf(fmaxf(v, 0.0f), 8191.0f);
  };
  for (int32_t i = threadIdx.x; i < p; i += blockDim.x) {
    unsigned long long k = ~0ull;
    if (i < m) {
      const double* r = M + 12 * (size_t)(base + i) + 8;  // z row
      const float f[4] = {(float)(r[0] * cx + r[1] * cy + r[2] * cz + r[3]), (float)(r[2] * ez),
                          (float)(r[0] * ex), (float)(r[1] * ey)};
      uint32_t q[4];
      for (int j = 0; j < 4; ++j) q[j] = quant(f[j]);
      unsigned long long code = 0;
      for (int b = 12; b >= 0; --b)
        for (int j = 0; j < 4; ++j) code = (code << 1) | ((q[j] >> b) & 1u);
      k = (code << 12) | (unsigned long long)i;  // 52-bit code, 12-bit index
    }
    key[i] = k;
  }
  __syncthreads();
  for (int32_t size = 2; size <= p; size <<= 1)
    for (int32_t stride = size >> 1; stride > 0; stride >>= 1) {
      for (int32_t i = threadIdx.x; i < p; i += blockDim.x) {
        const int32_t j = i ^ stride;
        if (j > i) {
          const bool up = (i & size) == 0;
          const unsigned long long a = key[i], b = key[j];
          if ((a > b) == up) {
            key[i] = b;
            key[j] = a;
          }
        }
      }
      __syncthreads();
    }
  for (int32_t i = threadIdx.x; i < m; i += blockDim.x) order[base + i] = (uint32_t)(base + (key[i] & 0xFFFu));
}

hipError_t launch_order_transforms(const double* M, int32_t n, int32_t fnx, int32_t fny, int32_t fnz, uint32_t* order,
                                   hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)((n + kOrderBlock - 1) / kOrderBlock);
  hipLaunchKernelGGL(order_transforms_kernel, dim3(blocks), dim3(1024), 0, s, M, n, 0.5f * (float)(fnx - 1),
                     0.5f * (float)(fny - 1), 0.5f * (float)(fnz - 1), (float)(fnx - 1), (float)(fny - 1),
                     (float)(fnz - 1), order);
  return hipGetLastError();
}

}  // namespace gemi
