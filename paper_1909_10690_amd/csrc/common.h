// Internal declarations shared by the HIP translation units of libgemi.so.
// Nothing here is part of the public ABI (include/gemi.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <math.h>
#include <stdint.h>

#include "plan.h"

namespace gemi {

// a * b + c with 24-bit unsigned operands (v_mad_u32_u24, full rate; a plain
// product may become the quarter-rate 64-bit multiply-add).
__device__ uint32_t mul24(uint32_t a, uint32_t b) __asm("llvm.amdgcn.mul.u24.i32");
__device__ __forceinline__ uint32_t mad24(uint32_t a, uint32_t b, uint32_t c) { return mul24(a, b) + c; }

constexpr int kMaxQ = 16;
constexpr int kBlock = 256;  // threads per workgroup of the reduction kernels (4 wave64)

// Entropic indices passed by value to the reduction kernels.
struct QList {
  double q[kMaxQ];
  int32_t n;
  int32_t pseudo;  // 1 = pseudo-additive Tsallis MI
};

// Exact floor(X / R) for 0 <= X < 2^24 as (X * m) >> s (Granlund and
// Montgomery, "Division by invariant integers using multiplication", PLDI
// 1994, Thm 4.2 with N = 24, l = ceil(log2 R), m = ceil(2^(N+l) / R)).
struct Divider {
  uint32_t m;
  uint32_t s;
};

inline Divider make_divider(uint32_t R) {
  uint32_t l = 0;
  while ((1u << l) < R) ++l;
  const uint64_t num = 1ull << (24 + l);
  Divider d;
  d.m = (uint32_t)((num + R - 1) / R);
  d.s = 24 + l;
  return d;
}

__device__ __forceinline__ uint32_t div_small(uint32_t x, Divider d) {
  return (uint32_t)(((uint64_t)x * d.m) >> d.s);
}

// Spacings and origins of a fixed/moving pair: voxel index i of a volume
// sits at origin + spacing * i (mm, per axis x, y, z).
struct Geometry {
  double fsp[3], forg[3];  // fixed
  double msp[3], morg[3];  // moving
};

// Index-space matrix M (fixed voxel index -> continuous moving index) of a
// physical fixed -> moving matrix P (Fig. 1 Transform block, mm):
//   M[r][c] = (P[r][c] * fsp[c]) / msp[r]                                        (c < 3)
//   M[r][3] = ((((P[r][0] forg[0] + P[r][1] forg[1]) + P[r][2] forg[2]) + P[r][3]) - morg[r]) / msp[r]
// one IEEE operation at a time in exactly this order, never fused, so that
// every implementation of the same definition quantises the same matrix.
__device__ __forceinline__ void compose_index_matrix(const double* __restrict__ P, const Geometry& g,
                                                     double* __restrict__ M) {
#pragma clang fp contract(off)
#pragma unroll
  for (int r = 0; r < 3; ++r) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double a = P[4 * r + c] * g.fsp[c];
      M[4 * r + c] = a / g.msp[r];
    }
    double o = P[4 * r] * g.forg[0];
    const double o1 = P[4 * r + 1] * g.forg[1];
    o = o + o1;
    const double o2 = P[4 * r + 2] * g.forg[2];
    o = o + o2;
    o = o + P[4 * r + 3];
    o = o - g.morg[r];
    M[4 * r + 3] = o / g.msp[r];
  }
}

// Q32 quantisation of one index-space 3x4 transform: Mq = rne(M * 2^32).
// A transform is usable when every entry is finite, linear entries are
// within +-2^16 and translations within +-2^24 (so that every coordinate of
// a volume of at most 4096 voxels per axis fits in int64).
__device__ __forceinline__ bool quantize_transform(const double* __restrict__ M, int64_t* Mq) {
  bool ok = true;
#pragma unroll
  for (int e = 0; e < 12; ++e) {
    const double m = M[e];
    const double lim = (e % 4 == 3) ? 16777216.0 : 65536.0;
    ok = ok && (fabs(m) <= lim);  // false for NaN and infinities
    Mq[e] = __double2ll_rn(m * 4294967296.0);
  }
  return ok;
}

// quantize_transform for a whole wave at once: lane e < 12 rounds entry e
// and the results are broadcast to scalar registers, with the same values
// and the same validity test.  Every lane of the wave takes part.
__device__ __forceinline__ bool quantize_transform_wave(const double* __restrict__ M, int64_t* Mq) {
  const int lane = threadIdx.x & 63;
  const int e = lane < 12 ? lane : 0;
  const double m = M[e];
  const double lim = (e % 4 == 3) ? 16777216.0 : 65536.0;
  const bool bad = lane < 12 && !(fabs(m) <= lim);  // true for NaN and infinities
  const int64_t v = __double2ll_rn(m * 4294967296.0);
  const uint32_t lo = (uint32_t)v, hi = (uint32_t)((uint64_t)v >> 32);
#pragma unroll
  for (int i = 0; i < 12; ++i)
    Mq[i] = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi, i) << 32) |
                      (uint32_t)__builtin_amdgcn_readlane(lo, i));
  return __builtin_amdgcn_ballot_w64(bad) == 0;
}

// A value every lane holds alike, moved to scalar registers.  A value
// computed by vector instructions stays in vector registers otherwise, and
// the compiler drops a readfirstlane builtin of a value it knows is uniform,
// so the value passes through an empty asm first, which hides that.  (Not the
// instruction itself in asm: gfx950 needs a wait state between a vector write
// and a v_readfirstlane of that register, and two before a vector instruction
// uses the scalar result; the compiler keeps these for its own instructions
// only, and where its code around the asm left none, a stale value was read.)
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  uint32_t lo = (uint32_t)v, hi = (uint32_t)((uint64_t)v >> 32);
  asm("" : "+v"(lo), "+v"(hi));
  return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(hi) << 32) |
                   (uint32_t)__builtin_amdgcn_readfirstlane(lo));
}

// ---------------------------------------------------------------------------
// per-voxel input preparation shared by the single-pair and multi-pair paths
// ---------------------------------------------------------------------------

// Fixed bin of an integer intensity: floor((clamp(u) - lo) * B / R).
__device__ __forceinline__ uint32_t fixed_bin_int(int32_t u, int32_t lo, int32_t hi, uint32_t bins,
                                                  Divider d) {
  u = u < lo ? lo : (u > hi ? hi : u);
  return div_small((uint32_t)(u - lo) * bins, d);
}

// Fixed bin of a float intensity: min(B-1, floor(((u - lo)/(hi - lo)) * B))
// in fp64, each step one IEEE operation.
__device__ __forceinline__ uint32_t fixed_bin_real(double u, double lo, double hi, int32_t bins) {
  u = u < lo ? lo : (u > hi ? hi : u);
  const double r = __ddiv_rn(__dsub_rn(u, lo), __dsub_rn(hi, lo));
  const int32_t b = (int32_t)floor(__dmul_rn(r, (double)bins));
  return (uint32_t)(b > bins - 1 ? bins - 1 : (b < 0 ? 0 : b));
}

// Clamped, offset intensity v' = clamp(v, lo, hi) - lo.
__device__ __forceinline__ uint32_t clamp_offset(int32_t v, int32_t lo, int32_t hi) {
  v = v < lo ? lo : (v > hi ? hi : v);
  return (uint32_t)(v - lo);
}

typedef unsigned int vec4u __attribute__((ext_vector_type(4)));
typedef unsigned int vec2u __attribute__((ext_vector_type(2)));

// Eight consecutive voxels at p (aligned to eight elements), clamped, offset
// and packed as 16-bit values: one load of 8 or 16 bytes.
__device__ __forceinline__ vec4u load_offset8(const __attribute__((address_space(1))) uint8_t* p, int32_t lo,
                                              int32_t hi) {
  const vec2u w = *(const __attribute__((address_space(1))) vec2u*)p;
  vec4u o;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t h = w[k >> 1] >> (16 * (k & 1));
    o[k] = clamp_offset((int32_t)(h & 0xFFu), lo, hi) | (clamp_offset((int32_t)((h >> 8) & 0xFFu), lo, hi) << 16);
  }
  return o;
}
template <typename T>
__device__ __forceinline__ vec4u load_offset8(const __attribute__((address_space(1))) T* p, int32_t lo, int32_t hi) {
  static_assert(sizeof(T) == 2, "u16 or i16");
  const vec4u w = *(const __attribute__((address_space(1))) vec4u*)p;
  vec4u o;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    o[k] = clamp_offset((int32_t)(T)(w[k] & 0xFFFFu), lo, hi) | (clamp_offset((int32_t)(T)(w[k] >> 16), lo, hi) << 16);
  return o;
}

// ---------------------------------------------------------------------------
// the fixed-volume sweep shared by the histogram kernels
// ---------------------------------------------------------------------------

// Maps workgroup id -> (transform, slab, band).  Workgroups are dealt
// round-robin to the 8 XCDs, so XCD x receives ids x, x+8, ...; those all
// take slabs from the x-th eighth of the fixed volume.  Slab-major order
// (within a band, when there are several) walks that eighth one thin slab
// at a time, all transforms per slab, so the workgroups resident on an XCD
// at once share one slab's moving footprint in that XCD's L2;
// transform-major order finishes a transform's slabs (all bands per slab)
// before the next transform.
__device__ __forceinline__ void block_work(int32_t chunks, int32_t n, int32_t bands,
                                           int32_t slab_major, uint32_t& t, uint32_t& chunk,
                                           uint32_t& band) {
  const uint32_t bid = blockIdx.x;
  const uint32_t xcd = bid & 7u, slot = bid >> 3;
  const uint32_t c8 = (uint32_t)chunks >> 3;
  const uint32_t nb = (uint32_t)bands;
  if (slab_major) {
    // bands slowest: every workgroup of band 0 is dispatched before any of
    // band 1, and so on.  A Parzen sweep's first band holds the background,
    // nearly every voxel of a CT, so its workgroups are the long ones:
    // dispatched first, they no longer trail the launch on a few CUs.
    const uint32_t per = c8 * (uint32_t)n;
    band = slot / per;
    const uint32_t rem = slot - band * per, cl = rem / (uint32_t)n;
    t = rem - cl * (uint32_t)n;
    chunk = xcd * c8 + cl;
  } else {
    const uint32_t per = c8 * nb;
    t = slot / per;
    const uint32_t rem = slot - t * per;
    band = rem / c8;
    chunk = xcd * c8 + (rem - band * c8);
  }
}

// Host-side launch descriptions.
struct VolumeDesc {
  const void* data;
  int32_t nx, ny, nz, dtype;
  double lo, hi;
};

// Geometry of one fixed/moving pair for the hard-binned sweep.
struct HardGeom {
  const uint8_t* fbins;  // fixed bins, [fnz][fny][fnx], rows in the sweep's FixedOrder
  const void* gvol;      // moving gather volume in layout `gather`
  int32_t fnx, fny, fnz;
  int32_t mnx, mny, mnz;
  uint32_t gvol_bytes;
  int32_t gather;        // Gather
  int32_t bins;
  Rods rods;     // of brick sweeps
  double scale;  // B / (R 2^48), R = moving hi - lo + 1
  Divider div;   // floor(X / R) for the exact fallback
};


struct HardLaunch {
  const double* transforms;  // [n][12]
  const uint8_t* fbins;      // fixed-volume bins, [fnz][fny][fnx], rows in the sweep's FixedOrder
  const void* gvol;          // moving gather volume in layout `gather` (Gather)
  VolumeDesc fixed, moving;
  uint32_t* hist;  // [n][B][B]
  uint64_t* count;  // [n]: each transform's sum of counts is added
  int32_t gather;
  int32_t n, bins, clamp;
  // workgroups per transform; [1] where choice[1] is not 0 (thin slabs; alike
  // where there is no choice)
  SlabSplit split[2];
  const uint32_t* choice;  // see Prepare, or NULL
  int32_t packed;  // 1: two 16-bit counters per LDS word (bins > 128)
  int32_t block;   // threads per workgroup: 256, 512 or 1024
  int32_t slab_major;  // workgroup order: 1 slab-major, 0 transform-major
  int32_t brick;       // 1: slabs as bricks of rods (RodWalk; 1024-thread launches)
  // processing order (launch_order_transforms), or NULL: the workgroups of
  // slot t sweep transform order[t] - order_t0; order_t0 is the batch index
  // of this launch's first transform
  const uint32_t* order;
  int64_t order_t0;
};

// Transforms per block of the processing order: the order is sorted within
// blocks of this many transforms, and launches that use it start at
// multiples of it.
constexpr int32_t kOrderBlock = 4096;

// The processing order of a batch of n index-space matrices for the hard
// sweep (order[i], absolute indices, a permutation of each block of
// kOrderBlock transforms): transforms whose images of the fixed volume lie
// at similar moving depths come together (see the kernel).
hipError_t launch_order_transforms(const double* M, int32_t n, int32_t fnx, int32_t fny, int32_t fnz, uint32_t* order,
                                   hipStream_t s);

// The gathers address their volume with 32-bit buffer offsets, so every
// gather volume stays below 4 GiB (the entry points check it).
constexpr size_t kMaxGatherBytes = 0xFFFFFFF0u;

// Bytes of the oct volume of an integer moving volume: per voxel the eight
// clamped, offset 16-bit corners of its 2x2x2 neighbourhood (16 bytes).
inline size_t oct_volume_bytes(int32_t nx, int32_t ny, int32_t nz) {
  return (size_t)nx * (size_t)ny * (size_t)nz * 16;
}

// The hard path packs 8-bit corners (8 bytes per voxel) when the moving
// range R = hi - lo + 1 is at most 256: the same single gather per voxel at
// half the bytes, which matters where the moving volumes stream from HBM.
inline bool oct8_range(double lo, double hi) { return hi - lo + 1.0 <= 256.0; }
inline size_t oct8_volume_bytes(int32_t nx, int32_t ny, int32_t nz) {
  return (size_t)nx * (size_t)ny * (size_t)nz * 8;
}

// Bytes of the plain 16-bit copy of an integer moving volume: the clamped,
// offset intensities u16[nz][ny][nx] and a pad of one slice, one row and two
// voxels (never more than the oct volume's bytes, whose region holds it).  A
// voxel's neighbourhood is four 32-bit loads, the pairs (x, x + 1) of rows y
// and y + 1 of slices z and z + 1; at the volume's upper faces these read
// past the row, slice or volume, where the weight is 0, so the pad needs no
// defined contents.  Float volumes on the sampled Parzen path: the same in
// fp32, with the pad set to 0.
inline size_t moving_copy_pad(int32_t nx, int32_t ny) { return (size_t)nx * ny + (size_t)nx + 2; }
inline size_t moving_copy_bytes(int32_t nx, int32_t ny, int32_t nz) {
  return ((size_t)nx * ny * (size_t)nz + moving_copy_pad(nx, ny)) * 2;
}

// Layouts of the hard sweeps' moving volume, and which one a call prepares:
// octs of 16-bit corners, or (kOctD, moving ranges of at most 2^14) of each
// row's difference and negated sum, from which a signed dot product forms the
// exact x-lerp in one instruction instead of two; octs of 8-bit corners; the
// plain copy.
// kTiled (brick sweeps): octs in tiles (tiled_index).
// kChoose (few transforms): the copy, or the octs, chosen on the device.
enum Gather : int32_t { kOct16 = 0, kOct8 = 1, kCopy16 = 2, kOctD = 3, kTiled = 4, kChoose = 8 };
__host__ __device__ constexpr int32_t gather_base(int32_t gather) { return gather & 3; }
__host__ __device__ constexpr int32_t gather_record(int32_t gather) {
  return gather_base(gather) == kOct8 ? 8 : (gather == kCopy16 ? 2 : 16);
}
inline size_t gather_volume_bytes(int32_t gather, int32_t nx, int32_t ny, int32_t nz) {
  if (gather == kCopy16) return moving_copy_bytes(nx, ny, nz);
  if (gather & kChoose) {
    const size_t copy = moving_copy_bytes(nx, ny, nz), octs = gather_volume_bytes(gather & ~kChoose, nx, ny, nz);
    return copy > octs ? copy : octs;
  }
  const bool rec8 = gather_base(gather) == kOct8;
  return (gather & kTiled ? tiled_records(nx, ny, nz, rec8) : (size_t)nx * ny * nz) * gather_record(gather);
}
// A gather instruction costs the texture unit about the same whatever its
// width, so a sweep over an oct volume (one gather per voxel) runs twice as
// fast as over the copy (four): 12.3 against 27.5 us a transform over a batch
// of 1000 of 256x256x180 u16.  But the oct volume is 8 times the moving
// volume to write and then to fetch, 36 us at that size against 8 us for the
// copy, so a call that prepares its volumes for a few transforms uses the
// copy (us a call, octs and copy, upright: 256x256x180 u16, 128 bins, one transform
// 112 and 73, two 127 and 98, four 168 and 146 -- but 220 and 307 turned by 30
// degrees, so beyond kCopyBytes only two; 128^3 u16, 64 bins, four 57 and 42).
// Turned, the copy's four gathers each have lines of their own, so such a
// call chooses on the device (turned_octs) -- a copy under kChooseBytes serves
// every turn: its lines stay in the L2s, and the choice costs a sweep 0.5 us (48^3).
constexpr int32_t kCopyTransforms = 4;
constexpr size_t kCopyBytes = 8 << 20, kChooseBytes = 1 << 20;
inline int32_t oct_gather(double lo, double hi) {
  return oct8_range(lo, hi) ? kOct8 : (hi - lo < 16384.0 ? kOctD : kOct16);
}
// room: bytes of the workspace's region for it.  Tiles of 16-byte records take
// longer to write than rows, 88 against 36 us at 256x256x180, which brick sweeps
// win back with about seven transforms (14 volumes of 128x128x48 to 512x512x200 in 5
// families of angles, mean of rows over tiles: four transforms 0.94, six 0.98, eight
// 1.01; us a call, tiles and rows, COMPACT_SLABS,
// 256x256x180 u16 turned up to +-20 degrees and by 0 to 90: two transforms 162 and
// 129, 166 and 146, four 234 and 205, 224 and 248, eight 284 and 288, 301 and 372);
// of 8-byte records no longer.
constexpr int32_t kRowsTransforms = 6;
inline int32_t hard_gather(const VolumeDesc& m, int32_t n, bool reused, bool brick, size_t room) {
  if (!reused && !brick) {
    const size_t copy = moving_copy_bytes(m.nx, m.ny, m.nz);
    if (n <= (copy > kCopyBytes ? 2 : kCopyTransforms))
      return copy > kChooseBytes ? oct_gather(m.lo, m.hi) | kChoose : (int32_t)kCopy16;
  }
  const int32_t oct = oct_gather(m.lo, m.hi);
  if (!reused && oct != kOct8 && n <= kRowsTransforms) return oct;
  return brick && gather_volume_bytes(oct | kTiled, m.nx, m.ny, m.nz) <= room ? oct | kTiled : oct;
}

// Whether such a call takes octs: what the copy's sweep costs more than the
// octs', over all its transforms, exceeds what the octs cost more to write.  With
// rho = min(|M[1][0]| / 2 + |M[2][0]|, 1), the rows a step along x rises by, and
// the voxels that lie inside, a transform's sweep costs about
// (inside / moving voxels) (0.3 + 1.7 rho^2) min(1.2, copy MB / 14) as much more as
// the octs cost to write: small copies stay in the L2s (us a call, copy and octs,
// turned by 0, 30, 60 and 90 degrees about y: 256x256x180 u16, one transform 73
// and 112, 111 and 118, 125 and 125, 166 and 138; two 98 and 127, 175 and 152, 212
// and 168, 246 and 184; 192^3, two 67 and 92, 106 and 110, 153 and 127, 216 and
// 132; 128^3, four 42 and 57, 60 and 60, 68 and 71, 101 and 73; 512x512x64, one, 83
// and 181, 68 and 155, 66 and 148, 77 and 151).  Octs of 8-bit corners cost 1.6 times
// less to write (256x256x180 u8, one transform, the same turns: 70 and 100, 108 and
// 104, 122 and 114, 154 and 122).  The weight of a voxel inside, 0 (the copy) where
// no turn can tip the choice by much:
inline float octs_weight(const VolumeDesc& f, const VolumeDesc& m, int32_t n) {
  const double mb = (double)moving_copy_bytes(m.nx, m.ny, m.nz) * 1e-6, small = mb / 14.0;
  const double vf = (double)f.nx * f.ny * f.nz, vm = (double)m.nx * m.ny * m.nz;
  const double w = (small < 1.2 ? small : 1.2) * vf / vm * (oct8_range(m.lo, m.hi) ? 1.6 : 1.0);
  return n * 2.0 * w > 1.5 ? (float)w : 0.0f;
}

// A batch of at most so many transforms on a moving volume whose octs take more
// bytes than that counts as turned or not, on the device (Prepare::choice[1]),
// and has a slab count for either (turned_slabs).
constexpr int32_t kTurnTransforms = 2;
constexpr size_t kTurnBytes = 64 << 20;
constexpr float kTurnedRise = 0.35f;  // mean |M[2][0]|; turned by 10 degrees the flat count is still the better one

// Bytes of the 16-bit quad volume of an integer moving volume on the Parzen
// path: per voxel the four (x, y) corners of its neighbourhood in one slice
// (clamped, offset values), one extra slice; two 8-byte loads per voxel at
// half the footprint of the oct volume, which matters when one transform's
// gathers cover a moving volume larger than the caches.
inline size_t quad16_bytes(int32_t nx, int32_t ny, int32_t nz) {
  return (size_t)nx * (size_t)ny * (size_t)(nz + 1) * 8;
}

// Bytes of the fp32 quad volume of a float moving volume: per voxel the
// four (x, y) corners of its neighbourhood in one slice, one extra slice.
inline size_t quad_f32_bytes(int32_t nx, int32_t ny, int32_t nz) {
  return (size_t)nx * (size_t)ny * (size_t)(nz + 1) * 16;
}

// The MI reduction splits each transform's table into reduce_splits(B, n)
// row slices (with the same-numbered columns' marginals), one workgroup
// each: a few transforms then still keep many CUs busy (1024 / n slices,
// at most B / 8 of >= 8 rows), while a large batch uses one workgroup per
// transform, whose per-workgroup overheads small slices would multiply.
// The slices' compensated partial sums are merged in slice order, so a
// result does not depend on scheduling; batches with the same slice count
// give bit-identical results for the same transform.
__host__ __device__ inline int32_t reduce_splits(int32_t bins, int64_t n) {
  if (bins < 16 || n <= 0) return 1;
  const int64_t s = 1024 / n;
  return (int32_t)(s < 1 ? 1 : (s > bins / 8 ? bins / 8 : s));
}

// Bytes of the partial sums: per transform, slice and entropy, three
// compensated (sum, error) pairs.
inline size_t reduce_part_bytes(int64_t n, int32_t bins, int32_t n_q) {
  return (size_t)n * reduce_splits(bins, n) * n_q * 3 * 16;
}

// Rows [r0, r1) of slice s of a B-row table split into S slices.
__host__ __device__ inline void slice_rows(int B, int S, int s, int& r0, int& r1) {
  r0 = (int)(((int64_t)B * s) / S);
  r1 = (int)(((int64_t)B * (s + 1)) / S);
}

struct ReduceLaunch {
  const uint32_t* hist;  // [n][B][B] counts, or NULL when `table` is used
  const double* table;   // [n][B][B] Parzen masses, or NULL
  uint64_t* count;       // [n] N < 2^28; the upper 32 bits are 0 before and after
  double* part;          // reduce_part_bytes(n, B, n_q) of partial sums
  const double* transforms;
  int32_t n, bins;
  int32_t splits;        // reduce_splits(bins, n), set by launch_mi_reduce
  double* marg_out;      // [n][2B] row then column marginals (masses), or NULL
  QList q;
  double* mi_out;        // [n][n_q]
  uint64_t* overlap_out; // [n] or NULL
};

// Parzen sweeps (see parzen.hip).
// Occupied fixed-bin rows of a Parzen call.  The Parzen sweeps index the
// table's rows by "slot" (rank among the occupied rows), so that the LDS
// bands cover only rows that hold voxels: a CT-like fixed volume occupies a
// few clusters of its bins (air, soft tissue, bone) and empty bands would
// still cost a full walk of the fixed volume each.
struct RowMap {
  uint32_t used[256];         // 1 for every bin some fixed voxel falls in
  uint32_t row_of_slot[256];  // table row of each slot
  uint32_t slot_of_row[256];  // slot of each occupied row
  uint32_t n_slots;           // occupied rows
};

struct ParzenArgs {
  const double* transforms;
  const uint8_t* fbins;       // fixed-volume slots (see RowMap)
  const RowMap* rows;
  const uint32_t* tile_mask;  // [row groups][x tiles]: slot groups present in each 16 x 4 wave tile
  const uint32_t* row_mask;   // [row groups]: the OR of each row group's tile masks
  const void* gvol;    // integer moving: 16-bit quads (full sweeps) or the 16-bit copy (sampled); float: f32 quads (sampled: f32 copy)
  double* table;       // [n][B][B] forward masses (fp64)
  uint64_t* count;     // [n] voxels that took part
  const float* gtab;   // [n][n_q][B][B] d MI / d p
  const double* marg;  // [n][2B] row then column marginals of the table (from the reduction)
  double* grad;        // [n][n_q][12]
  int32_t fnx, fny, fnz;
  int32_t mnx, mny, mnz;
  uint32_t gvol_bytes;
  int32_t n, bins, chunks, bands, band_rows, slab_major;
  const uint32_t* records;  // sampled: see launch_sample_layout, or NULL (the copy)
  int32_t n_q, q0;     // backward: entropies [q0, q0 + NQG) of n_q
  float sscale;        // (B - 4) / (hi - lo)
  double dsdv;         // (B - 4) / (hi - lo), fp64
};

constexpr int kParzenQGroup = 2;  // entropies per backward sweep

// Wave tiles of the Parzen walks (kTileX x kTileY fixed voxels, one wave
// step): bit g of a tile's mask is set when a voxel of the tile has a slot
// in [8 g, 8 g + 8).  A band's walk skips the tiles whose mask holds none
// of its slots, so every band but the background's skips the background.
constexpr int kSlotGroup = 8;
inline int64_t parzen_tiles(int32_t nx, int32_t ny, int32_t nz) {
  return (int64_t)((ny + kTileY - 1) / kTileY) * nz * ((nx + kTileX - 1) / kTileX);
}
// Row groups (kTileY rows of one slice): each also gets the OR of its
// tiles' masks, stored after the tile masks, so that a band's walk skips a
// row group without any of its slots in one test (in a CT nearly every
// voxel is background, so the other bands find their slots in a fifth of
// the row groups and a few percent of the tiles).
inline int64_t parzen_row_groups(int32_t ny, int32_t nz) { return (int64_t)((ny + kTileY - 1) / kTileY) * nz; }
__host__ __device__ inline uint32_t slot_group_mask(int32_t r_lo, int32_t r_hi) {
  const int32_t g0 = r_lo / kSlotGroup, g1 = (r_hi - 1) / kSlotGroup;  // r_hi > r_lo
  return (g1 >= 31 ? 0xFFFFFFFFu : ((2u << g1) - 1u)) & ~((1u << g0) - 1u);
}

// Forward sweeps: the background row (slot 0, the lowest occupied fixed
// bin: air in a CT) receives most voxels, all into a few cells.  Its first
// parzen_hot_cols(B) columns get kHotCopies private copies in LDS, lane l
// adding into copy l % kHotCopies; each copy is one cell longer than the
// columns it covers, so the same column of consecutive copies falls in
// different LDS banks.
constexpr int kHotCopies = 16;
// Row pitch (cells) of the Parzen sweeps' LDS tables: the band's B columns
// and a pad of 3, so that one column of consecutive rows falls 3 (fp32
// cells) or 6 (64-bit cells) banks apart, not in one bank as with a pitch
// of B (a multiple of 32 words for the usual bin counts).
__host__ __device__ inline int32_t parzen_pitch(int32_t bins) { return bins + 3; }
constexpr int kHotCols = 64;
__host__ __device__ inline int32_t parzen_hot_cols(int32_t bins) { return bins < kHotCols ? bins : kHotCols; }
__host__ __device__ inline int32_t parzen_hot_stride(int32_t bins) { return parzen_hot_cols(bins) + 1; }
__host__ __device__ inline int32_t parzen_hot_cells(int32_t bins) { return kHotCopies * parzen_hot_stride(bins); }


struct ParzenLaunch {
  ParzenArgs args;
  int32_t float_quads;  // 1: moving volume is fp32 (float4 quads)
  int32_t clamp;
  int32_t block;        // threads per workgroup of the sweeps: 256, 512 or 1024
};

// LDS guard of every launch with dynamic LDS: the kernel's static LDS (read
// once with hipFuncGetAttributes) plus `dynamic` must fit the device's
// per-workgroup maximum, and `dynamic` the maximum the kernel was
// configured for (hipErrorInvalidValue otherwise; nothing is launched).
// lds_register() records a kernel's static LDS and the device maximum at
// configuration; lds_guard() looks up kernels it has not seen.
hipError_t lds_register(const void* kernel);
// at_zero: the kernel addresses its dynamic LDS from address 0, so it must
// keep no static LDS.
hipError_t lds_guard(const void* kernel, size_t dynamic, size_t configured_max, bool at_zero = false);

// Up to kMax arrays to zero (4-byte aligned, whole words).
struct ClearList {
  static constexpr int32_t kMax = 5;
  uint32_t* p[kMax] = {};
  size_t words[kMax] = {};
  int32_t n = 0;
  void add(void* q, size_t bytes) {
    if (bytes == 0) return;
    p[n] = (uint32_t*)q;
    words[n++] = bytes / 4;
  }
};
// d MI / d P from d MI / d M in place, rows of 12 (gradients of `rows`
// transform-entropy pairs): G_P[r][c] = (G_M[r][c] fsp[c] + G_M[r][3] forg[c]) / msp[r],
// G_P[r][3] = G_M[r][3] / msp[r].
hipError_t launch_grad_physical(double* grad, int64_t rows, const Geometry& g, hipStream_t s);
// The order of a fixed volume's bins: voxel order, or that the thin-slab
// (fixed_run_x) or brick (cube_run_x) sweeps read.
enum FixedOrder : int32_t { kVoxelOrder = 0, kRunOrder = 1, kCubeOrder = 2 };
template <int ORDER>
__host__ __device__ constexpr int32_t stored_x(int32_t p, int32_t nx) {
  return ORDER == kRunOrder ? fixed_run_x(p, nx) : (ORDER == kCubeOrder ? cube_run_x(p, nx) : p);
}
// The bins in voxel order; used[256], if given (zeroed before), gets a 1 for
// every bin that some voxel falls in.
hipError_t launch_prebin_voxels(const VolumeDesc& f, int bins, uint8_t* out, uint32_t* used, hipStream_t s);

// What a call does before its sweep, in one launch; each part only if given.
struct Prepare {
  // index-space matrices M[n][12] of the caller's physical matrices P[n][12]
  const double* P = nullptr;
  double* M = nullptr;
  int64_t n = 0;
  Geometry geo = {};
  ClearList clear;
  // the fixed volume's bins, in an order of FixedOrder
  uint8_t* fbins = nullptr;
  VolumeDesc f = {};
  int32_t bins = 0, order = 0;
  // the integer moving volume in layout `gather`
  void* gvol = nullptr;
  VolumeDesc m = {};
  int32_t gather = 0;
  // kCopy16 only: where *records is not 0, octs (kOct16) instead
  const uint32_t* records = nullptr;
  // What the device chooses (n <= kCopyTransforms): [0] 1 where a kChoose volume is
  // octs (written with it), [1] 1 where the transforms are turned (written with M)
  uint32_t* choice = nullptr;
  float weight = 0.0f;  // octs_weight
  int32_t clamp = 0;
};
// Layout of a sampled Parzen call's moving volume, chosen on the device, where
// the matrices are: *records = 1 (octs; float volumes: quads) where the mean
// over the batch (at most 256 matrices of it, evenly spaced) of the rows a step
// along x rises by, row_weight |M[1][0]| + |M[2][0]|, exceeds `limit`, else 0
// (the plain copy).  P: physical matrices.
hipError_t launch_sample_layout(const double* P, int64_t n, const Geometry& g, double row_weight, double limit,
                                uint32_t* records, hipStream_t s);
hipError_t launch_prepare(const Prepare& p, hipStream_t s);
// Nothing is written where `records` is given and *records is not 0 (copy) or 0
// (quads).
hipError_t launch_pack_copy_f32(const VolumeDesc& m, float* out, hipStream_t s, const uint32_t* records = nullptr);
hipError_t launch_hist_hard(const HardLaunch& L, hipStream_t s);
// Random subsampling (sample.hip): the kept fixed voxels as list entries
// {x | y << 12 | fixed bin << 24, z}; n_list must be zero beforehand.
hipError_t launch_sample_list(const uint8_t* fbins, int32_t nx, int32_t ny, int32_t nz, double fraction,
                              uint64_t seed, uint2* list, unsigned long long* n_list, hipStream_t s);
hipError_t launch_hist_sampled(const HardLaunch& L, const uint2* list, const unsigned long long* n_list,
                               hipStream_t s);

// Many fixed/moving pairs of uneven sizes (see pairs.hip).
struct PairDesc {
  const void* fixed;
  const void* moving;
  const double* transforms;  // caller's [n_t][12], physical
  Geometry geo;              // the pair's spacings and origins
  HardGeom geom;             // fbins / octs point into the workspace
  int32_t fdtype, mdtype;
  double flo, fhi;           // fixed range (fp64 rule for float fixed volumes)
  int32_t mlo, mhi;          // moving range
  Divider fdiv;              // floor(X / R_fixed)
  int32_t n_t, chunks;       // transforms, slabs (a multiple of 8)
};

// Pairs' preparation, one wave per item: chunks of consecutive stored bytes
// of a fixed volume, of consecutive records of a moving volume (16 per lane).
constexpr int kPrepLane = 16, kPrepChunk = 64 * kPrepLane;

struct PairsArgs {
  const PairDesc* pairs;
  int32_t n_pairs;
  const int64_t* fchunk_base;  // [P+1] prefix of kPrepChunk-voxel chunks of the fixed volumes
  const int64_t* mchunk_base;  // [P+1] prefix of kPrepChunk-record chunks of the moving volumes
  const int64_t* t_base;     // [P+1] prefix of transforms
  const int64_t* xcd_base;   // [8][P+1] prefix of work items per XCD
  unsigned long long* counters;  // [8] work-queue heads
  double* transforms;        // [T][12], gathered and composed to index space
  uint32_t* hist;            // [T][B][B]
  uint64_t* count;           // [T]: sums of the counts
  int32_t bins;
  int32_t transform_major;   // work-item order within a pair: 0 slab-major, 1 transform-major
};

struct PairsLaunch {
  PairsArgs args;
  int64_t total_t, fixed_chunks, moving_chunks;
  int32_t clamp, packed, cu_count;
  int32_t block;  // threads per workgroup of the sweep: 256, 512 or 1024
  int32_t gather;  // layout of every pair's moving volume
};

// The transforms gathered and composed; with `volumes` also the pairs'
// fixed bins and oct volumes.
hipError_t launch_pairs_prep(const PairsLaunch& L, hipStream_t s, bool volumes = true);
hipError_t launch_pairs_hist(const PairsLaunch& L, hipStream_t s);
HardGeom make_hard_geom(const VolumeDesc& fixed, const VolumeDesc& moving, const uint8_t* fbins,
                        const void* gvol, int32_t gather, int32_t bins);
hipError_t launch_mi_reduce(const ReduceLaunch& L, hipStream_t s);
hipError_t launch_pack_quads_f32(const VolumeDesc& m, float4* out, hipStream_t s, const uint32_t* records = nullptr);
hipError_t launch_pack_quads16(const VolumeDesc& m, uint2* out, hipStream_t s);
// The row map of m->used, the fixed bins turned into slots in place, and the
// tile and row group masks (see kSlotGroup).
hipError_t launch_slots(uint8_t* fbins, int32_t nx, int32_t ny, int32_t nz, int32_t bins, RowMap* m, uint32_t* mask,
                        hipStream_t s);
hipError_t launch_parzen_fwd(const ParzenLaunch& L, hipStream_t s);
hipError_t launch_parzen_sampled_fwd(const ParzenLaunch& L, const uint2* list, const unsigned long long* n_list,
                                     hipStream_t s);
hipError_t launch_dmi_dp(const ParzenLaunch& L, const QList& q, hipStream_t s);
hipError_t launch_parzen_bwd(const ParzenLaunch& L, hipStream_t s);
hipError_t launch_lds_atomic_probe(uint32_t* out, int32_t blocks, int32_t iters, hipStream_t s);

}  // namespace gemi
