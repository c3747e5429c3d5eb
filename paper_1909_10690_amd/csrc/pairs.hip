// Hard-binned MI of many fixed/moving pairs of uneven sizes, each with its
// own transforms, in one persistent launch (the batched evaluation behind
// the exhaustive per-family sweeps of the Methodology, for many volumes).
//
// Work items are (pair, slab, transform) triples.  Each pair's slabs are
// split into 8 equal shares, one per XCD, and every XCD has its own work
// queue: a workgroup (resident for the whole launch) repeatedly takes the
// next item of its XCD's queue with one atomic, sweeps that slab for that
// transform into its LDS histogram, adds the histogram into the
// transform's HBM histogram and clears it.  Items are ordered pair-major,
// then slab-major, so the workgroups of an XCD work on one slab of one pair
// at a time and share its moving footprint in L2.  A slab is a compact brick
// of rods (RodWalk), swept as sweep_rods has it.  What bounds the sweep is
// the vector unit, at about 46 instructions a wave step of 64 samples, with
// the L1's line fills behind: 24 pairs of 64^3 to 256^3 voxels, 16 rigid
// transforms each, 64 bins: 2068 us a sweep with bricks of whole x rows over
// untiled octs, 2283 with rods over untiled octs, 1885 with rods over tiles.
// Every workgroup leaves the loop once its queue is empty, so the grid
// always drains.
//
// Per-pair fixed bins and moving octs are prepared by two kernels over the
// items of all pairs (runs of 1024 stored bytes, runs of 1024 records), one
// wave per item, and the transforms are gathered into one array for the MI
// reduction.
#include "common.h"
#include "sweep.h"

namespace gemi {

// Largest p with base[p] <= v, for base[0] = 0 <= v < base[P].
__device__ __forceinline__ int find_pair(const int64_t* __restrict__ base, int P, int64_t v) {
  int lo = 0, hi = P;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (base[mid] <= v)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// Device-memory views: the pairs' volume pointers are read from the pair
// table, so without the address space the compiler would use flat accesses.
typedef const __attribute__((address_space(1))) uint16_t global_u16;
typedef const __attribute__((address_space(1))) int16_t global_i16;
typedef const __attribute__((address_space(1))) uint4_t global_cu4;
typedef const __attribute__((address_space(1))) float global_f32;
typedef __attribute__((address_space(1))) uint8_t global_out8;
typedef __attribute__((address_space(1))) uint32_t global_out32;
typedef __attribute__((address_space(1))) uint2_t global_out2;
typedef __attribute__((address_space(1))) uint4_t global_out4;

__device__ __forceinline__ int32_t load_int(const void* p, int32_t dtype, size_t i) {
  switch (dtype) {
  case 0: return ((global_u8*)p)[i];
  case 1: return ((global_u16*)p)[i];
  default: return ((global_i16*)p)[i];
  }
}

__global__ void gather_transforms_kernel(PairsArgs a, int64_t total) {
  for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < total;
       g += (int64_t)gridDim.x * blockDim.x) {
    const int p = find_pair(a.t_base, a.n_pairs, g);
    const double* src = a.pairs[p].transforms + 12 * (g - a.t_base[p]);
    double M[12];
    compose_index_matrix(src, a.pairs[p].geo, M);
    for (int e = 0; e < 12; ++e) a.transforms[12 * g + e] = M[e];
  }
}

// A value every lane holds alike, moved to scalar registers.  The work item
// reaches the workgroup through LDS, so the compiler cannot tell that what is
// derived from it is uniform: without the broadcast the pair's geometry stays
// in vector registers, is reloaded inside the sweep, and each gather from the
// moving volume runs a loop over the distinct buffer descriptors of the wave.
template <typename T>
__device__ __forceinline__ T uniform(const T& v) {
  static_assert(sizeof(T) % 4 == 0, "32-bit words");
  uint32_t w[sizeof(T) / 4];
  __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 4; ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
  T r;
  __builtin_memcpy(&r, w, sizeof(T));
  return r;
}

// Calls f(d, item, lane) for the items of the concatenated item space
// [base[0], base[P]) that fall to this workgroup, d being the descriptor of
// the item's pair and item its index within the pair: a contiguous range
// per workgroup, one wave per item.  The pair is found once per wave and
// then advanced as the items ascend; its bounds and descriptor are loaded
// again only when it changes (they come through vector loads, so a load
// per item would put two dependent round trips before every item's data).
template <typename F>
__device__ __forceinline__ void for_each_item(const PairDesc* __restrict__ pairs,
                                              const int64_t* __restrict__ base, int P, int64_t items,
                                              F&& f) {
  const int64_t per = (items + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = (int64_t)blockIdx.x * per;
  const int64_t r1 = r0 + per < items ? r0 + per : items;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int lane = threadIdx.x & 63;
  if (r0 + wave >= r1) return;
  int p = uniform(find_pair(base, P, r0 + wave));
  int64_t lo = uniform(base[p]), hi = uniform(base[p + 1]);
  PairDesc d = uniform(pairs[p]);
  for (int64_t r = r0 + wave; r < r1; r += nw) {
    if (r >= hi) {
      do {
        ++p;
        lo = hi;
        hi = uniform(base[p + 1]);
      } while (r >= hi);
      d = uniform(pairs[p]);
    }
    f(d, r - lo, lane);
  }
}

// The bins of 16 consecutive voxels at src (16-byte aligned), a whole run of a
// row, in stored order: stored byte 4 j + k is voxel 4 k + j.
template <typename T, typename F>
__device__ __forceinline__ uint4_t run_bins(const __attribute__((address_space(1))) T* src, F&& bin) {
  constexpr int W = (int)sizeof(T);  // 16-byte words of the run
  uint4_t v[W];
#pragma unroll
  for (int i = 0; i < W; ++i) v[i] = ((global_cu4*)src)[i];
  uint4_t o;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t b = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int e = 4 * k + j, per = 16 / W;  // voxels a 16-byte word
      const uint32_t word = v[e / per][(e % per) * W / 4];
      T u;
      if constexpr (W == 4) u = __builtin_bit_cast(T, word);
      else u = (T)(word >> (8 * ((e * W) & 3)));
      b |= bin(u) << (8 * k);
    }
    o[j] = b;
  }
  return o;
}

// Fixed bins of every pair in the sweep's order (cube_run_x), one wave per
// chunk of kPrepChunk consecutive stored bytes of a pair's fixed volume:
// every lane busy whatever the row length.  Full chunks of aligned volumes
// whose rows are whole runs (nx a multiple of 16) are handled a run per lane,
// in 16-byte accesses (2 pairs of 256^3 u16: 57 us a byte per lane at a time, 20
// now); otherwise lane l takes bytes l, l + 64, ..., the row of each found from
// the one before.
__global__ void prep_fixed_kernel(PairsArgs a, int64_t chunks) {
  for_each_item(a.pairs, a.fchunk_base, a.n_pairs, chunks, [&](const PairDesc& d, int64_t c, int lane) {
    const int64_t nvox = (int64_t)d.geom.fnx * d.geom.fny * d.geom.fnz;
    const int64_t c0 = c * kPrepChunk;
    global_out8* __restrict__ out = (global_out8*)d.geom.fbins;
    auto bin_int = [&](int32_t u) {
      return fixed_bin_int(u, (int32_t)d.flo, (int32_t)d.fhi, (uint32_t)d.geom.bins, d.fdiv);
    };
    auto bin_real = [&](float u) { return fixed_bin_real((double)u, d.flo, d.fhi, d.geom.bins); };
    if (d.geom.fnx % kCubeRun == 0 && c0 + kPrepChunk <= nvox && (((uintptr_t)d.fixed | (uintptr_t)out) & 15) == 0) {
      const int64_t at = c0 + kPrepLane * lane;
      uint4_t o;
      switch (d.fdtype) {  // the same for every lane
      case 0: o = run_bins((global_u8*)d.fixed + at, bin_int); break;
      case 1: o = run_bins((global_u16*)d.fixed + at, bin_int); break;
      case 2: o = run_bins((global_i16*)d.fixed + at, bin_int); break;
      default: o = run_bins((global_f32*)d.fixed + at, bin_real);
      }
      *(global_out4*)(out + at) = o;
      return;
    }
    const uint32_t nx = (uint32_t)d.geom.fnx;
    uint32_t p = (uint32_t)c0 + (uint32_t)lane;  // < 2^28
    uint32_t base = p / nx * nx, x = p - base;   // the row's first voxel, the place in the row
    for (int k = 0; k < kPrepLane && p < (uint32_t)nvox; ++k) {
      const uint32_t v = base + (uint32_t)cube_run_x((int32_t)x, (int32_t)nx);
      out[p] = (uint8_t)(d.fdtype == 3 ? bin_real(((global_f32*)d.fixed)[v]) : bin_int(load_int(d.fixed, d.fdtype, v)));
      p += 64;
      x += 64;
      if (x >= nx) {
        const uint32_t rows = nx >= 64 ? 1 : x / nx;
        base += rows * nx;
        x -= rows * nx;
      }
    }
  });
}

// The voxels x .. x + 4 (8-bit) or x .. x + 3 (16-bit) of the row whose voxel x
// lies at index at, past the row's end its last one again (left: voxels of the
// row from x on).  Loads at any address; at the volume's end they start earlier,
// so that they stay within.
template <typename T>
__device__ __forceinline__ uint64_t row_words(const void* vol, uint32_t at, uint32_t left, uint32_t nvox) {
  const uint32_t from = at + 4 <= nvox ? at : nvox - 4;  // nvox >= 8
  if constexpr (sizeof(T) == 1) {
    global_u8* const p = (global_u8*)vol;
    uint32_t v = *(global_unaligned32*)(p + from) >> (8 * (at - from));
    const uint32_t end = p[at + (left > 4 ? 4u : left - 1)];
    if (left < 4) v = (v & ((1u << (8 * left)) - 1)) | ((end * 0x01010101u) << (8 * left));
    return v | ((uint64_t)end << 32);
  } else {
    uint64_t v = *(global_unaligned64*)((global_u8*)vol + 2 * (size_t)from) >> (16 * (at - from));
    if (left < 4) {
      const uint64_t keep = (1ull << (16 * left)) - 1, last = (v >> (16 * (left - 1))) & 0xFFFFu;
      v = (v & keep) | ((last * 0x0001000100010001ull) & ~keep);
    }
    return v;
  }
}

// Moving oct volumes of every pair, with the layout and clamping of the
// single-pair path, one wave per chunk of kPrepChunk consecutive records.
// In tiles, a lane takes the records of one tile row (4 of 8 bytes, or 2 of 16),
// 32 bytes, so that a wave's stores are 2 KiB of consecutive records, from one
// or two loads of each of its four source rows (2 pairs of 256^3 u16: 214 us,
// with a load a corner 271; u8: 94 us with a 4-byte and a 1-byte load a row, 106
// with one of 8 bytes).  Untiled, or 16-bit voxels in 8-bit
// corners: a record per lane at a time.
__global__ void prep_moving_kernel(PairsArgs a, int64_t items) {
  for_each_item(a.pairs, a.mchunk_base, a.n_pairs, items, [&](const PairDesc& d, int64_t c, int lane) {
    const uint32_t nx = (uint32_t)d.geom.mnx, ny = (uint32_t)d.geom.mny, nz = (uint32_t)d.geom.mnz;
    const uint32_t plane = nx * ny, nvox = plane * nz;
    const int32_t base = gather_base(d.geom.gather);
    const bool tiled = (d.geom.gather & kTiled) != 0, o8 = base == kOct8;
    const uint32_t px = (uint32_t)tile_pad_x((int32_t)nx, o8), py = (uint32_t)tile_pad((int32_t)ny);
    const uint32_t records = d.geom.gvol_bytes / (o8 ? 8u : 16u);  // < 2^32
    const uint32_t c0 = (uint32_t)c * kPrepChunk;
    // Tile rows: REC records of a row to a lane; f(records' first index, the
    // four source rows from voxel x on).
    auto tile_rows = [&]<typename T, uint32_t REC>(auto&& f) {
      const uint32_t tx = px / REC, ty = py / 2;
#pragma unroll
      for (uint32_t k = 0; k < kPrepChunk / (64 * REC); ++k) {
        const uint32_t i = c0 + 64 * REC * k + REC * (uint32_t)lane;
        if (i >= records) break;
        const uint32_t tile = i / (4 * REC), tr = tile / tx, tz = tr / ty;
        uint32_t y = (tr - tz * ty) * 2 + (lane & 1), z = tz * 2 + ((lane >> 1) & 1);
        y = y < ny ? y : ny - 1;  // padding: any defined contents
        z = z < nz ? z : nz - 1;
        const uint32_t x = (tile - tr * tx) * REC;  // < nx
        const uint32_t at = z * plane + y * nx + x, dy = y + 1 < ny ? nx : 0, dz = z + 1 < nz ? plane : 0;
        const uint64_t rows[4] = {row_words<T>(d.moving, at, nx - x, nvox), row_words<T>(d.moving, at + dy, nx - x, nvox),
                                  row_words<T>(d.moving, at + dz, nx - x, nvox),
                                  row_words<T>(d.moving, at + dz + dy, nx - x, nvox)};
        f(i, rows);
      }
    };
    if (tiled && o8 && d.mdtype == 0) {
      const bool ident = d.mlo == 0 && d.mhi == 255;  // 8-bit corners: the clamp changes nothing then
      tile_rows.template operator()<uint8_t, 4>([&](uint32_t i, const uint64_t (&rows)[4]) {
        uint32_t w[4], e[4];  // voxels x .. x + 3 and x + 4 of each source row
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          w[r] = (uint32_t)rows[r];
          e[r] = (uint32_t)(rows[r] >> 32) & 0xFFu;
          if (!ident) {
            uint32_t o = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) o |= clamp_offset((int32_t)((w[r] >> (8 * b)) & 0xFFu), d.mlo, d.mhi) << (8 * b);
            w[r] = o;
            e[r] = clamp_offset((int32_t)e[r], d.mlo, d.mhi);
          }
        }
        // records: byte 4 dz + 2 dy + dx' (layout of pack_oct8)
        auto pair = [&](int r, int j) -> uint32_t {  // bytes j, j + 1 of row r
          return j < 3 ? (w[r] >> (8 * j)) & 0xFFFFu : (w[r] >> 24) | (e[r] << 8);
        };
        uint4_t o[2];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          o[j >> 1][2 * (j & 1)] = pair(0, j) | (pair(1, j) << 16);
          o[j >> 1][2 * (j & 1) + 1] = pair(2, j) | (pair(3, j) << 16);
        }
        global_out4* __restrict__ out = (global_out4*)((global_out2*)d.geom.gvol + i);
        out[0] = o[0];
        out[1] = o[1];
      });
      return;
    }
    if (tiled && !o8) {
      auto records2 = [&]<typename T>() {
        tile_rows.template operator()<T, 2>([&](uint32_t i, const uint64_t (&rows)[4]) {
          uint4_t o[2];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            uint32_t v[3];
#pragma unroll
            for (int b = 0; b < 3; ++b)
              v[b] = clamp_offset((int32_t)(T)(rows[r] >> (8 * sizeof(T) * b)), d.mlo, d.mhi);
            o[0][r] = v[0] | (v[1] << 16);
            o[1][r] = v[1] | (v[2] << 16);
          }
          global_out4* __restrict__ out = (global_out4*)d.geom.gvol + i;
          out[0] = o[0];
          out[1] = o[1];
        });
      };
      switch (d.mdtype) {  // the same for every lane
      case 0: records2.template operator()<uint8_t>(); break;
      case 1: records2.template operator()<uint16_t>(); break;
      default: records2.template operator()<int16_t>();
      }
      return;
    }
    auto val = [&](size_t i) -> uint32_t { return clamp_offset(load_int(d.moving, d.mdtype, i), d.mlo, d.mhi); };
    const uint32_t kx = o8 ? 4 : 2;  // tile width
    for (uint32_t k = 0; k < kPrepLane; ++k) {
      const uint32_t out = c0 + 64 * k + (uint32_t)lane;
      if (out >= records) break;
      uint32_t x, y, z;
      if (tiled) {
        const uint32_t tile = out / (4 * kx), low = out - tile * (4 * kx);
        const uint32_t tr = tile / (px / kx), tz = tr / (py / 2);
        x = (tile - tr * (px / kx)) * kx + low % kx;
        y = (tr - tz * (py / 2)) * 2 + low / kx % 2;
        z = 2 * tz + low / (2 * kx);
        if (x >= nx || y >= ny || z >= nz) continue;  // padding: never gathered
      } else {
        const uint32_t row = out / nx;
        x = out - row * nx;
        z = row / ny;
        y = row - z * ny;
      }
      const uint32_t v = z * plane + y * nx + x;
      const uint32_t dx = x + 1 < nx ? 1 : 0, dy = y + 1 < ny ? nx : 0, dz = z + 1 < nz ? plane : 0;
      if (o8) {
        ((global_out2*)d.geom.gvol)[out] =
            uint2_t{val(v) | (val(v + dx) << 8) | (val(v + dy) << 16) | (val(v + dy + dx) << 24),
                    val(v + dz) | (val(v + dz + dx) << 8) | (val(v + dz + dy) << 16) | (val(v + dz + dy + dx) << 24)};
      } else {
        ((global_out4*)d.geom.gvol)[out] =
            uint4_t{val(v) | (val(v + dx) << 16), val(v + dy) | (val(v + dy + dx) << 16),
                    val(v + dz) | (val(v + dz + dx) << 16), val(v + dz + dy) | (val(v + dz + dy + dx) << 16)};
      }
    }
  });
}

template <bool CLAMP, bool PACKED, int GL, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(8))) void hist_pairs_kernel(PairsArgs a) {
  extern __shared__ uint32_t lds_hist[];
  const int B = a.bins;
  const int words = B * hist_row_words(B, PACKED);
  // the work-item slot follows the histogram in the dynamic LDS (the sweep
  // addresses the histogram from LDS address 0: no static LDS)
  int64_t& item_sh = *(int64_t*)(lds_hist + ((words + 1) & ~1));
  clear_hist<PACKED, NT>(lds_hist, B);
  const uint32_t xcd = blockIdx.x & 7u;
  const int64_t* __restrict__ xbase = a.xcd_base + (int64_t)xcd * (a.n_pairs + 1);
  const int64_t total = xbase[a.n_pairs];
  // The items a workgroup takes from its queue ascend, so its pair only
  // moves forward: the pair's bounds, geometry and counts are loaded again
  // only when an item falls past it (a search per item put about log2 P
  // dependent loads before every slab's sweep).
  int p = -1;
  int64_t p_lo = 0, p_hi = 0;  // xbase[p], xbase[p + 1]; xbase[0] = 0
  HardGeom geom;
  int32_t n_t = 0, chunks = 0;
  int64_t t0 = 0;
  for (;;) {
    if (threadIdx.x == 0) item_sh = (int64_t)atomicAdd(&a.counters[xcd], 1ull);
    __syncthreads();
    const int64_t item = uniform(item_sh);
    if (item >= total) break;  // the same for every thread of the workgroup
    if (item >= p_hi) {
      do {  // item < total = xbase[P] bounds p + 1 <= P
        ++p;
        p_lo = p_hi;
        p_hi = uniform(xbase[p + 1]);
      } while (item >= p_hi);
      geom = uniform(a.pairs[p].geom);
      n_t = uniform(a.pairs[p].n_t);
      chunks = uniform(a.pairs[p].chunks);
      t0 = uniform(a.t_base[p]);
    }
    const int64_t rem = item - p_lo;
    // slab-major items: one slab's transforms in a row (the slab's moving
    // footprint stays in L2); transform-major: a transform's slabs in a row
    int64_t slab, tl;
    if (a.transform_major) {
      const int64_t per = chunks >> 3;
      tl = rem / per;
      slab = rem - tl * per;
    } else {
      slab = rem / n_t;
      tl = rem - slab * n_t;
    }
    const uint32_t chunk = xcd * (uint32_t)(chunks >> 3) + (uint32_t)slab;
    const int64_t t = t0 + tl;
    const double* Md = a.transforms + 12 * t;
    int64_t Mq[12];
    const bool ok = quantize_transform(Md, Mq);  // (the wave-parallel form measured 0.8% slower here)
    if (ok) {
      int64_t Ms[12];
#pragma unroll
      for (int e = 0; e < 12; ++e) Ms[e] = uniform64(Mq[e]);
      sweep_rods<CLAMP, PACKED, GL, NT / 64>(geom, Md, Ms, chunks, chunk, lds_hist);
    }
    __syncthreads();
    if (ok) flush_hist<PACKED, NT>(lds_hist, B, a.hist + (size_t)t * B * B, a.count + t, true);
    __syncthreads();
  }
}

// Workgroups (4 waves each) for a preparation kernel: a few per CU, fewer
// for small item counts.
static unsigned row_grid(int64_t rows) {
  const int64_t g = (rows + 3) / 4;
  return (unsigned)(g < 4096 ? (g > 0 ? g : 1) : 4096);
}

hipError_t launch_pairs_prep(const PairsLaunch& L, hipStream_t s, bool volumes) {
  if (L.total_t > 0) {
    const int64_t blocks = (L.total_t + 255) / 256;
    hipLaunchKernelGGL(gather_transforms_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)),
                       dim3(256), 0, s, L.args, L.total_t);
  }
  if (!volumes) return hipGetLastError();
  if (L.fixed_chunks > 0)
    hipLaunchKernelGGL(prep_fixed_kernel, dim3(row_grid(L.fixed_chunks)), dim3(256), 0, s, L.args,
                       L.fixed_chunks);
  if (L.moving_chunks > 0)
    hipLaunchKernelGGL(prep_moving_kernel, dim3(row_grid(L.moving_chunks)), dim3(256), 0, s, L.args,
                       L.moving_chunks);
  return hipGetLastError();
}

// Dynamic LDS limit of the pairs sweep (a u32 table up to 128 bins, 16-bit
// pairs above, and the work-item slot after it).
constexpr size_t kPairsLdsMax = 150 * 1024;

template <bool CLAMP, bool PACKED, int GL, int NT>
static hipError_t pairs_variant(const PairsLaunch& L, hipStream_t s) {
  const int B = L.args.bins;
  const size_t words = (size_t)B * hist_row_words(B, PACKED);
  const size_t lds = ((words + 1) & ~(size_t)1) * 4 + 8;  // histogram, then the 8-byte item slot
  const void* fn = (const void*)hist_pairs_kernel<CLAMP, PACKED, GL, NT>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kPairsLdsMax);
  if (e != hipSuccess || (e = lds_guard(fn, lds, kPairsLdsMax, true)) != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, NT, lds);
  if (e != hipSuccess) return e;
  if (per_cu < 1) per_cu = 1;
  // every queue needs workgroups: a multiple of 8 (one share per XCD)
  const unsigned grid = (unsigned)(((per_cu * L.cu_count + 7) / 8) * 8);
  hipLaunchKernelGGL((hist_pairs_kernel<CLAMP, PACKED, GL, NT>), dim3(grid), dim3(NT), lds, s, L.args);
  return hipGetLastError();
}

template <bool CLAMP, bool PACKED, int GL>
static hipError_t pairs_block(const PairsLaunch& L, hipStream_t s) {
  switch (L.block) {
  case 256: return pairs_variant<CLAMP, PACKED, GL, 256>(L, s);
  case 1024: return pairs_variant<CLAMP, PACKED, GL, 1024>(L, s);
  default: return pairs_variant<CLAMP, PACKED, GL, 512>(L, s);
  }
}

template <int GL>
static hipError_t pairs_layout(const PairsLaunch& L, hipStream_t s) {
  if (L.clamp) return L.packed ? pairs_block<true, true, GL>(L, s) : pairs_block<true, false, GL>(L, s);
  return L.packed ? pairs_block<false, true, GL>(L, s) : pairs_block<false, false, GL>(L, s);
}

hipError_t launch_pairs_hist(const PairsLaunch& L, hipStream_t s) {
  switch (L.gather) {
  case kOct8 | kTiled: return pairs_layout<kOct8 | kTiled>(L, s);
  case kOct16 | kTiled: return pairs_layout<kOct16 | kTiled>(L, s);
  case kOct8: return pairs_layout<kOct8>(L, s);
  case kOct16: return pairs_layout<kOct16>(L, s);
  default: return hipErrorInvalidValue;
  }
}

}  // namespace gemi
