// The hard-binned histogram sweep of one slab of the fixed volume for one
// transform, shared by the single-pair kernel (hard.hip) and the persistent
// multi-pair kernel (pairs.hip).  Internal to libgemi.so.
#pragma once

#include "common.h"

#pragma clang fp contract(off)

namespace gemi {

typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
typedef short short2_t __attribute__((ext_vector_type(2)));
typedef unsigned int uint2_t __attribute__((ext_vector_type(2)));
typedef unsigned int uint4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uint32_t lds_u32;
// Device-memory bytes: loads through such a pointer are global, not flat,
// also when the pointer itself was read from memory.
typedef const __attribute__((address_space(1))) uint8_t global_u8;
typedef uint32_t unaligned32 __attribute__((aligned(1)));
typedef const __attribute__((address_space(1))) unaligned32 global_unaligned32;
typedef uint64_t unaligned64 __attribute__((aligned(1)));
typedef const __attribute__((address_space(1))) unaligned64 global_unaligned64;

// Loads of one record of a buffer whose descriptor has a stride: the
// hardware forms base + index * stride, so the index needs no shift.
__device__ uint4_t struct_load_b128(__amdgpu_buffer_rsrc_t rsrc, int vindex, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.struct.ptr.buffer.load.v4i32");
__device__ uint2_t struct_load_b64(__amdgpu_buffer_rsrc_t rsrc, int vindex, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.struct.ptr.buffer.load.v2i32");
__device__ uint32_t struct_load_b32(__amdgpu_buffer_rsrc_t rsrc, int vindex, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.struct.ptr.buffer.load.i32");

// v0 (1 - w) + v1 w at 16-bit weight w = fx >> 16, exact: the pair's low
// half times (65535 - w), high half times w, plus the low half once more.
__device__ __forceinline__ uint32_t lerp_x(uint32_t pair, uint32_t wpack) {
  return __builtin_amdgcn_udot2(__builtin_bit_cast(ushort2_t, pair),
                                __builtin_bit_cast(ushort2_t, wpack), pair & 0xFFFFu, false);
}

// The same from a record word -(v0 + v1) | (v1 - v0) << 16 (kOctD), with
// `weights` -2^15 low and w - 2^15 high:
// (v0 + v1) 2^15 + (v1 - v0) (w - 2^15) = v0 (2^16 - w) + v1 w, one signed dot
// product (below 2^30: the clamp changes nothing, and keeps the compiler from
// the accumulating form, whose register it would have to clear first).
__device__ __forceinline__ uint32_t lerp_xd(uint32_t rec, uint32_t weights) {
  return (uint32_t)__builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, rec), __builtin_bit_cast(short2_t, weights), 0,
                                          true);
}

// (float)(q >> 16): one instruction (the compiler shifts and converts).
__device__ __forceinline__ float high16_f32(uint32_t q) {
  float f;
  asm("v_cvt_f32_u32_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1" : "=v"(f) : "v"(q));
  return f;
}

// Exact bin of V = sum over corners, from the four exact x-lerps.
static __device__ __noinline__ uint32_t exact_bin(uint32_t a00, uint32_t a10, uint32_t a01, uint32_t a11,
                                           uint32_t wy, uint32_t wz, uint32_t B, Divider div) {
  const uint64_t b0 = (uint64_t)a00 * (65536u - wy) + (uint64_t)a10 * wy;
  const uint64_t b1 = (uint64_t)a01 * (65536u - wy) + (uint64_t)a11 * wy;
  const uint64_t V = b0 * (65536u - wz) + b1 * wz;
  // floor(V B / (R 2^48)) = floor(X / R), X = floor(V B / 2^48) < 2^24
  const uint32_t X = (uint32_t)(V >> 48) * B + (uint32_t)(((V & 0xFFFFFFFFFFFFull) * B) >> 48);
  return div_small(X, div);
}

// The bin of a hard sweep is read off an fp32 value and redone in integers
// where rounding could matter.  With p = V B / (R 2^48) < B the exact bin
// position, the sweep forms u = kBinBase + p + 4 ulp (ulp: that of u, 2^-16 for
// kBinBase = 128, up to 128 bins; 2^-15 for 256, above).  V comes from the four
// exact x-lerps with five roundings on sums of non-negative terms (to float,
// a product and an fma per axis), the scale is rounded once and u once, so
// |error| <= 6 2^-24 p + ulp / 2 <= 3.5 ulp (p < kBinBase).  So the integer
// part of u is the bin when its fraction is at least 8 ulp; otherwise (1.2e-4
// of positions, 2.4e-4 above 128 bins, and those exactly on an edge)
// exact_bin decides.
constexpr uint32_t kBinGuard = 8;  // ulp
// kBinBase + 4 ulp; 16-bit counters take any bin count, u32 ones at most 128
constexpr float bin_base(bool packed) { return (packed ? 256.0f : 128.0f) * (1.0f + 4.0f / 8388608.0f); }

// Per-launch constants of the hard-binned step of one fixed voxel: the
// moving gather volume, its upper coordinates, the bin scale and the LDS
// histogram's row pitch.
struct HardStep {
  __amdgpu_buffer_rsrc_t rsrc;
  uint64_t topx, topy, topz;
  uint32_t NY, MX, Bu, row_bytes, row_cells;
  float scale;     // B / (R 2^48)
  uint32_t shift2;  // 2, in a vector register
  Divider div;

  int32_t to_row, to_slice;  // kCopy16: bytes to the next row, next slice
  uint32_t ny2, mx2, low_y, low_z;  // kTiled: the constants of tiled_index

  // gather: the layout the kernel's GL instance reads
  __device__ __forceinline__ HardStep(const HardGeom& g, bool packed, int32_t gather) {
    topx = (uint64_t)(g.mnx - 1) << 32;
    topy = (uint64_t)(g.mny - 1) << 32;
    topz = (uint64_t)(g.mnz - 1) << 32;
    NY = (uint32_t)g.mny;
    MX = (uint32_t)g.mnx;
    // records of 16, 8 or 2 bytes, indexed by voxel; the record bound is
    // given in bytes, which is no tighter than any record count
    rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)g.gvol, (short)gather_record(gather), (int)g.gvol_bytes, 0x00020000);
    to_row = 2 * g.mnx;
    to_slice = 2 * g.mnx * g.mny;
    const bool rec8 = gather_base(gather) == kOct8;
    const uint32_t s = rec8 ? 4u : 2u, px = (uint32_t)tile_pad_x(g.mnx, rec8), py = (uint32_t)tile_pad(g.mny);
    ny2 = py / 2;
    mx2 = 2 * px;
    low_y = mx2 - s;
    low_z = px * py - 2 * s;  // < 2^24
    Bu = (uint32_t)g.bins;
    // LDS histogram row pitch: in bytes (u32 counters), in 16-bit cells
    // (packed counters)
    row_bytes = 4u * (uint32_t)hist_row_words(g.bins, false);
    row_cells = 2u * (uint32_t)hist_row_words(g.bins, true);
    scale = (float)g.scale;
    shift2 = 2;
    asm("" : "+v"(shift2));
    div = g.div;
  }

  // Counts one fixed voxel whose exact Q32 moving coordinates (qx, qy, qz)
  // are given: clamped (CLAMP) or skipped when outside [0, n - 1] on any
  // axis; fixed_bin() supplies its fixed bin (read after the gather is
  // issued).  CHECK false: the caller has established that the voxel lies
  // inside on every axis, where clamping and skipping change nothing.
  template <bool CLAMP, bool PACKED, int GL, bool CHECK = true, typename FB>
  __device__ __forceinline__ void count(int64_t qx, int64_t qy, int64_t qz, FB&& fixed_bin,
                                        uint32_t* lds_hist) const {
    uint64_t cx = (uint64_t)qx, cy = (uint64_t)qy, cz = (uint64_t)qz;
    if (!CHECK) {
    } else if (CLAMP) {
      cx = qx < 0 ? 0 : (cx > topx ? topx : cx);
      cy = qy < 0 ? 0 : (cy > topy ? topy : cy);
      cz = qz < 0 ? 0 : (cz > topz ? topz : cz);
    } else {
      // 0 <= q <= top; a negative q wraps to a huge unsigned value
      if (cx > topx || cy > topy || cz > topz) return;
    }
    const uint32_t ix = (uint32_t)(cx >> 32), iy = (uint32_t)(cy >> 32), iz = (uint32_t)(cz >> 32);
    // rows iz ny + iy < ny nz <= 2^24 and edges <= 4096: 24-bit operands
    uint32_t vox;
    if (GL & kTiled)  // tiled_index
      vox = mad24(mad24(iz, ny2, iy), mx2, 4 * ix) -
            mad24(iz & 1u, low_z, mad24(iy & 1u, low_y, 3u * (ix & (gather_base(GL) == kOct8 ? 3u : 1u))));
    else
      vox = mad24(mad24(iz, NY, iy), MX, ix);
    const uint32_t fx = (uint32_t)cx, fy = (uint32_t)cy, fz = (uint32_t)cz;
    uint32_t a00, a10, a01, a11;  // the exact x-lerps of the four rows
    if (gather_base(GL) == kOctD) {
      const uint4_t oc = struct_load_b128(rsrc, (int)vox, 0, 0, 0);
      const uint32_t w = (fx & 0xFFFF0000u) ^ 0x80008000u;
      a00 = lerp_xd(oc.x, w);
      a10 = lerp_xd(oc.y, w);
      a01 = lerp_xd(oc.z, w);
      a11 = lerp_xd(oc.w, w);
    } else {
      uint4_t oc;
      if (gather_base(GL) == kOct8) {
        // bytes (x,y), (x1,y), (x,y1), (x1,y1) of slice z in .x, of z1 in .y
        const uint2_t d = struct_load_b64(rsrc, (int)vox, 0, 0, 0);
        oc.x = __builtin_amdgcn_perm(0u, d.x, 0x0C010C00u);  // (b0, b1) as 16-bit halves
        oc.y = __builtin_amdgcn_perm(0u, d.x, 0x0C030C02u);  // (b2, b3)
        oc.z = __builtin_amdgcn_perm(0u, d.y, 0x0C010C00u);
        oc.w = __builtin_amdgcn_perm(0u, d.y, 0x0C030C02u);
      } else if (GL == kCopy16) {
        oc.x = struct_load_b32(rsrc, (int)vox, 0, 0, 0);
        oc.y = struct_load_b32(rsrc, (int)vox, 0, to_row, 0);
        oc.z = struct_load_b32(rsrc, (int)vox, 0, to_slice, 0);
        oc.w = struct_load_b32(rsrc, (int)vox, 0, to_slice + to_row, 0);
      } else {
        oc = struct_load_b128(rsrc, (int)vox, 0, 0, 0);
      }
      // (65535 - wx) in the low half, wx in the high half: the high halves of
      // ~fx and fx, one byte permute
      const uint32_t wpack = __builtin_amdgcn_perm(fx, ~fx, 0x07060302u);
      a00 = lerp_x(oc.x, wpack);
      a10 = lerp_x(oc.y, wpack);
      a01 = lerp_x(oc.z, wpack);
      a11 = lerp_x(oc.w, wpack);
    }
    // the moving bin: y- and z-lerps, scale and base in fp32 (see kBinGuard)
    const float wy = high16_f32(fy), wz = high16_f32(fz);
    const float uy = 65536.0f - wy, uz = 65536.0f - wz;
    const float b0 = fmaf((float)a10, wy, (float)a00 * uy);
    const float b1 = fmaf((float)a11, wy, (float)a01 * uy);
    const float u = fmaf(fmaf(b1, wz, b0 * uz), scale, bin_base(PACKED));
    // bits 16..22 (PACKED: doubled, 16..23) hold the bin, the low 16 bits the
    // fraction
    const uint32_t bits = PACKED ? 2u * __builtin_bit_cast(uint32_t, u) : __builtin_bit_cast(uint32_t, u);
    // one 16-bit compare and a branch of the whole wave; the lanes concerned
    // are looked for behind it
    constexpr uint32_t guard = PACKED ? 2u * kBinGuard : kBinGuard;
    uint64_t near_edge;
    asm("v_cmp_gt_u16_e64 %0, %1, %2" : "=s"(near_edge) : "n"(guard), "v"(bits));
    auto exact = [&](uint32_t& cell, uint32_t shift) {
      uint32_t b = bits;
      asm volatile("" : "+v"(b));
      if ((b & 0xFFFFu) < guard) cell = exact_bin(a00, a10, a01, a11, fy >> 16, fz >> 16, Bu, div) << shift;
    };
    const uint32_t fb = fixed_bin();
    if (PACKED) {
      // 16-bit cell of counter [fb][bm]; the row pitch is even, so the
      // cell's word and half follow from it directly
      uint32_t bm = (bits >> 16) & 0xFFu;
      if (near_edge != 0) exact(bm, 0);
      const uint32_t cell = __umul24(fb, row_cells) + bm;
      atomicAdd(&lds_hist[cell >> 1], 1u << ((cell & 1u) * 16u));
    } else {
      // LDS byte address of counter [fb][bm], formed directly: byte 2 of u
      // (up to 128 bins bit 23, the exponent's last, is 0) shifted in one
      // instruction, and a multiply-add.  The kernels that sweep keep no
      // static LDS, so their dynamic histogram starts at address 0 (lds_guard
      // checks this at launch) and needs no base.
      uint32_t bm4;
      asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2"
          : "=v"(bm4)
          : "v"(shift2), "v"(bits));
      if (near_edge != 0) exact(bm4, 2);
      const uint32_t addr = mad24(fb, row_bytes, bm4);
      __hip_atomic_fetch_add((lds_u32*)(size_t)addr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
};

// The x ranges of a wave's row groups (range_lane, range_value, row_spans):
// lanes 0..15 hold the bound constants of the transform, and each row group
// takes the least v of each group of four lanes with two quad permutes.
struct RowRanges {
  RangeLane c;
  bool exact;  // uniform: every lane's constants exact

  // Md: the transform's 12 entries (index space, row-major 3 x 4) in device
  // memory; each lane reads its axis row and rounds it to Q32 as
  // quantize_transform does.
  __device__ __forceinline__ void init(const double* Md, const HardGeom& g, int lane) {
    const int a = (lane & 3) == 3 ? 0 : (lane & 3);
    const double* row = Md + 4 * a;
    const double q = 4294967296.0;
    const double m0 = __builtin_rint(row[0] * q), m1 = __builtin_rint(row[1] * q);
    const double m2 = __builtin_rint(row[2] * q), m3 = __builtin_rint(row[3] * q);
    const int32_t n = a == 0 ? g.mnx : (a == 1 ? g.mny : g.mnz);
    c = range_lane(lane, m0, m1, m2, m3, (double)(n - 1) * q);
    exact = __builtin_amdgcn_ballot_w64(!c.exact) == 0;
  }

  // Spans of the row group at (j0, k); the whole wave takes part.
  __device__ __forceinline__ RowSpans spans(int32_t j0, int32_t k, int32_t full, bool skip) const {
    if (!exact) return RowSpans{0, full, full, full};
    int32_t v = range_value(c, j0, k);
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false));  // quad_perm 1,0,3,2
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false));  // quad_perm 2,3,0,1
    return row_spans(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 4),
                     __builtin_amdgcn_readlane(v, 8), __builtin_amdgcn_readlane(v, 12), full, skip);
  }
};

// Sweeps one thin slab of the fixed volume for one transform (Mq) into the
// workgroup's LDS histogram.  NW waves share the slab's 4-row groups.
// GL: the moving volume's layout (Gather); kOct8 corners (one 64-bit gather)
// are unpacked into the 16-bit pairs of the x-lerp with byte permutes.
// Md: the transform as stored; Mq: its Q32 rounding, in scalar registers
// (quantize_transform_wave).
template <bool CLAMP, bool PACKED, int GL, int NW>
__device__ __forceinline__ void sweep_hard(const HardGeom& g, const double* Md, const int64_t* Mq,
                                           const SlabSplit& split, uint32_t chunk, uint32_t* lds_hist) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int dx = lane & (kTileX - 1), dy = lane / kTileX;
  // the matrix in scalar registers (quantize_transform_wave puts it there):
  // the walk's row coordinates and steps are then scalar values, and only
  // the lane offsets take vector registers
  const int64_t* M = Mq;
  GroupWalk w;
  w.init(M, g.fny, g.fnz, split.slabs, chunk, wave, NW, dx, dy, false, split.slab_nz);
  const int64_t sx = w.step[0], sy = w.step[1], sz = w.step[2];
  const HardStep hs(g, PACKED, GL);
  // Fixed bins: the row's address in scalar registers, the lane's offset in a
  // vector register.  Every load, however narrow, costs the texture unit as
  // much as the moving gather, so the bins come four x steps to a 32-bit load:
  // in each whole 64-voxel run of a row they are stored in the order
  // fixed_run_x.
  const uint32_t fnx = (uint32_t)g.fnx;
  global_u8* const fbins = (global_u8*)g.fbins;
  const uint32_t lane_f = dy * fnx + dx, lane_f4 = dy * fnx + 4 * dx;
  const int32_t full = (int32_t)(fnx / kTileX);      // x steps every lane of the tile takes
  const int32_t runs = (int32_t)(fnx / kFixedRun) * (kFixedRun / kTileX);  // of these, in whole runs
  const bool tail = (uint32_t)dx < fnx % kTileX;  // the lane takes one more
  const bool has_tail = fnx % kTileX != 0;
  RowRanges ranges;
  ranges.init(Md, g, lane);

  for (; w.g < w.g1; w.next()) {
    // x steps [c0, c1) have every lane inside; with EXCLUDE no lane counts
    // outside [u0, u1)
    const RowSpans sp = ranges.spans(w.j0, w.k, full, !CLAMP);
    const int32_t j = w.j0 + dy;
    if (j >= g.fny) continue;
    global_u8* const row = fbins + ((uint32_t)w.k * (uint32_t)g.fny + (uint32_t)w.j0) * fnx;  // < 2^28
    int64_t qx = w.r[0] + w.lane_off[0], qy = w.r[1] + w.lane_off[1], qz = w.r[2] + w.lane_off[2];
    if (sp.u0 > 0) {
      qx += sx * sp.u0;
      qy += sy * sp.u0;
      qz += sz * sp.u0;
    }
    // whole runs with every lane inside, four x steps at a time: [c0, c1)
    const int32_t c0 = (sp.c0 + 3) & ~3, c1 = (sp.c1 < runs ? sp.c1 : runs) & ~3;
    int32_t it = sp.u0;
    uint32_t bins4 = 0;  // the lane's bins of steps it, it + 1, ... of the run
    auto load_run = [&] { return *(global_unaligned32*)(row + (uint32_t)(it >> 2) * kFixedRun + lane_f4); };
    auto checked = [&](int32_t end) {
      if ((it & 3) != 0 && it < runs) bins4 = load_run() >> (8 * (it & 3));  // a start within a run
      for (; it < (end < runs ? end : runs); ++it, bins4 >>= 8, qx += sx, qy += sy, qz += sz) {
        if ((it & 3) == 0) bins4 = load_run();
        hs.count<CLAMP, PACKED, GL>(qx, qy, qz, [&] { return bins4 & 0xFFu; }, lds_hist);
      }
    };
    if (c0 < c1) {
      checked(c0);
      for (; it < c1; it += 4) {
        bins4 = load_run();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          hs.count<CLAMP, PACKED, GL, false>(qx, qy, qz, [&] { return (bins4 >> (8 * k)) & 0xFFu; }, lds_hist);
          qx += sx;
          qy += sy;
          qz += sz;
          asm("" : "+v"(qx), "+v"(qy), "+v"(qz));  // step by step: not each from the first, with twice the adds
        }
      }
    }
    checked(sp.u1);
    for (; it < sp.u1; ++it, qx += sx, qy += sy, qz += sz)  // past the last whole run
      hs.count<CLAMP, PACKED, GL>(
          qx, qy, qz, [&] { return (uint32_t)row[(uint32_t)it * kTileX + lane_f]; }, lds_hist);
    if (has_tail && tail) {
      qx = w.r[0] + sx * full + w.lane_off[0];
      qy = w.r[1] + sy * full + w.lane_off[1];
      qz = w.r[2] + sz * full + w.lane_off[2];
      hs.count<CLAMP, PACKED, GL>(qx, qy, qz, [&] { return (uint32_t)row[(uint32_t)full * kTileX + lane_f]; }, lds_hist);
    }
  }
}

// Sweeps one brick of the fixed volume (RodWalk) for one transform into the
// workgroup's LDS histogram; arguments as sweep_hard.  For transforms that
// rotate widely: a wave's 64 voxels are a cube, whose moving image touches
// about half the cache lines of a 16 x 4 tile's whichever way it is turned, and
// with tiled octs (kTiled) half of those again -- the sweep is bound by the
// lines its gathers touch and fetch (729 rotations of up to 180 degrees,
// 256x256x180 u16 at 128 bins: 36.8 ms with 16 x 4 tiles in bricks of whole x
// rows, 18.6 with rods and tiles).  Each wave classes its rod by the extreme
// coordinates over the rod: outside the moving volume on some axis (skipped
// when EXCLUDE), inside on all (no test per voxel), or mixed.
template <bool CLAMP, bool PACKED, int GL, int NW>
__device__ __forceinline__ void sweep_rods(const HardGeom& g, const double* Md, const int64_t* Mq, int32_t chunks,
                                           uint32_t chunk, uint32_t* lds_hist) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const Rods rods = g.rods;
  const int dx = lane & 3, dy = (lane >> 2) & (rods.ry() - 1), dz = lane >> (2 + rods.ly);
  const HardStep hs(g, PACKED, GL);
  const int64_t sx = 4 * Mq[0], sy = 4 * Mq[4], sz = 4 * Mq[8];
  const int64_t ox = Mq[0] * dx + Mq[1] * dy + Mq[2] * dz;
  const int64_t oy = Mq[4] * dx + Mq[5] * dy + Mq[6] * dz;
  const int64_t oz = Mq[8] * dx + Mq[9] * dy + Mq[10] * dz;
  // lane a < 3: the matrix row of axis a, the least and greatest offsets over
  // a rod and the upper coordinate
  const int axis = lane < 3 ? lane : 0;
  const double* mrow = Md + 4 * axis;
  const int64_t m0 = __double2ll_rn(mrow[0] * 4294967296.0), m1 = __double2ll_rn(mrow[1] * 4294967296.0);
  const int64_t m2 = __double2ll_rn(mrow[2] * 4294967296.0), m3 = __double2ll_rn(mrow[3] * 4294967296.0);
  const int64_t ex = m0 * (rods.longest(g.fnx) - 1), ey = m1 * (rods.ry() - 1), ez = m2 * (rods.rz() - 1);
  const int64_t omin = (ex < 0 ? ex : 0) + (ey < 0 ? ey : 0) + (ez < 0 ? ez : 0);
  const int64_t omax = (ex > 0 ? ex : 0) + (ey > 0 ? ey : 0) + (ez > 0 ? ez : 0);
  const int64_t top = (int64_t)((axis == 0 ? g.mnx : (axis == 1 ? g.mny : g.mnz)) - 1) << 32;
  const uint32_t fnx = (uint32_t)g.fnx, fplane = fnx * (uint32_t)g.fny;
  const uint32_t lane_f = dz * fplane + dy * fnx + dx, lane_f4 = lane_f + 3 * dx;
  global_u8* const fbins = (global_u8*)g.fbins;
  RodWalk w;
  w.init(rods, g.fny, g.fnz, chunks, chunk, wave);
  for (; w.u < w.u1; w.next(NW)) {
    const int32_t x0 = w.x0(), j0 = w.j0(), k0 = w.k0();
    const int64_t r = m0 * x0 + m1 * j0 + m2 * k0 + m3;
    // lanes past axis 2 repeat axis 0
    const bool inside = __builtin_amdgcn_ballot_w64(r + omin < 0 || r + omax > top) == 0;
    if (!CLAMP && __builtin_amdgcn_ballot_w64(r + omax < 0 || r + omin > top) != 0) continue;
    auto lane_value = [&](int a) {
      return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)((uint64_t)r >> 32), a) << 32) |
                       (uint32_t)__builtin_amdgcn_readlane((uint32_t)r, a));
    };
    int64_t qx = lane_value(0) + ox, qy = lane_value(1) + oy, qz = lane_value(2) + oz;
    if (j0 + dy >= g.fny || k0 + dz >= g.fnz) continue;
    global_u8* const rod = fbins + ((uint32_t)k0 * fplane + (uint32_t)j0 * fnx + (uint32_t)x0);  // < 2^28
    const int32_t width = w.xs == rods.segments - 1 ? g.fnx - x0 : rods.width;
    const int32_t runs = width / kCubeRun;  // whole runs of 16 voxels, four steps each
    for (int32_t run = 0; run < runs; ++run) {
      const uint32_t bins4 = *(global_unaligned32*)(rod + (uint32_t)run * kCubeRun + lane_f4);
      auto steps = [&]<bool CHECK>() {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          hs.template count<CLAMP, PACKED, GL, CHECK>(qx, qy, qz, [&] { return (bins4 >> (8 * k)) & 0xFFu; }, lds_hist);
          qx += sx;
          qy += sy;
          qz += sz;
          asm("" : "+v"(qx), "+v"(qy), "+v"(qz));  // step by step: not each from the first, with twice the adds
        }
      };
      if (inside)
        steps.template operator()<false>();
      else
        steps.template operator()<true>();
    }
    for (int32_t x = runs * kCubeRun; x < width; x += 4, qx += sx, qy += sy, qz += sz)  // the rest of the row
      if (x + dx < width)
        hs.count<CLAMP, PACKED, GL>(qx, qy, qz, [&] { return (uint32_t)rod[(uint32_t)x + lane_f]; }, lds_hist);
  }
}

// Clears a workgroup's LDS histogram, padding included (16-byte stores,
// then the last words).
template <bool PACKED, int NT>
__device__ __forceinline__ void clear_hist(uint32_t* lds_hist, int B) {
  const int words = B * hist_row_words(B, PACKED), quads = words >> 2;
  uint4_t* q = (uint4_t*)lds_hist;
  for (int e = threadIdx.x; e < quads; e += NT) q[e] = uint4_t{0u, 0u, 0u, 0u};
  for (int e = (quads << 2) + (int)threadIdx.x; e < words; e += NT) lds_hist[e] = 0;
}

// Adds the non-zero LDS bins into a transform's HBM histogram [B][B] (and
// clears them for the next use of the LDS histogram when `rezero`): a wave
// per fixed-bin row at a time, a lane per counter word.
// A row holds at most 256 counter words (B <= 256), four per lane, so each
// row is unrolled into four fixed chunks whose addresses differ from the
// first by immediate offsets.
// The counts' sum is added to *count, by one atomic per call: the waves' sums
// meet in a padding word of the first row, which is 0 before and after.
template <bool PACKED, int NT>
__device__ __forceinline__ void flush_hist(uint32_t* lds_hist, int B, uint32_t* __restrict__ out,
                                           uint64_t* __restrict__ count, bool rezero) {
  const int pitch = hist_row_words(B, PACKED), used = PACKED ? (B + 1) / 2 : B;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  uint32_t sum = 0;
  for (int r = wave; r < B; r += NT / 64) {
    uint32_t* __restrict__ row = out + (size_t)r * B;
    uint32_t* src = lds_hist + r * pitch;
    uint32_t vs[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) vs[c] = lane + 64 * c < used ? src[lane + 64 * c] : 0u;  // reads issued together
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int w = lane + 64 * c;
      const uint32_t v = vs[c];
      if (v == 0) continue;
      if (rezero) src[w] = 0;
      if (PACKED) {
        sum += (v & 0xFFFFu) + (v >> 16);
        if (v & 0xFFFFu) atomicAdd(&row[2 * w], v & 0xFFFFu);
        if (v >> 16) atomicAdd(&row[2 * w + 1], v >> 16);  // never set past the row's last bin
      } else {
        sum += v;
        atomicAdd(&row[w], v);
      }
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
  if (lane == 0 && sum) atomicAdd(&lds_hist[used], sum);
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t all = lds_hist[used];
    if (all) atomicAdd((unsigned long long*)count, (unsigned long long)all);
    lds_hist[used] = 0;
  }
}

}  // namespace gemi
