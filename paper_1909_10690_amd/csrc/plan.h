// Launch-planning arithmetic of libgemi.so: pure host functions with no HIP
// dependency, shared by the launchers and compiled on its own by the CPU
// unit test of the planning rules.  Internal; not part of the public ABI.
#pragma once

#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include <initializer_list>

namespace gemi {

// A dispatch counts its work-items in 32 bits: a grid of n x (workgroups
// per transform) x threads beyond that wraps without an error and leaves
// transforms unevaluated.  Every launcher whose grid grows with the number
// of transforms issues launches of whole transforms, each below 2^31
// work-items.
constexpr int64_t kMaxWorkItemsPerLaunch = 0x7FFFFFFF;

// Transforms per launch for a kernel of `workgroups_per_transform`
// workgroups of `threads` threads (at least 1).
inline int32_t transforms_per_launch(int64_t workgroups_per_transform, int32_t threads) {
  const int64_t per = workgroups_per_transform * threads;
  const int64_t m = per > 0 ? kMaxWorkItemsPerLaunch / per : 1;
  return (int32_t)(m < 1 ? 1 : (m > 0x7FFFFFFF ? 0x7FFFFFFF : m));
}

// Workgroups of 256 threads for n items, one a thread (beyond 8192 workgroups
// in turns).
constexpr uint32_t fill_blocks(size_t n) {
  const size_t g = (n + 255) / 256;
  return (uint32_t)(g > 8192 ? 8192 : (g < 1 ? 1 : g));
}

// Row parts of a volume (256 voxels of a row each, fewer at a row's end; at most
// 2^24), and the workgroups of 256 threads that take them: one each up to 2^22,
// in turns beyond, because a workgroup for each of 2^24 would wrap a launch.
constexpr uint32_t row_parts(int32_t nx, int32_t ny, int32_t nz) {
  return (((uint32_t)nx + 255) / 256) * (uint32_t)ny * (uint32_t)nz;
}
constexpr uint32_t row_part_blocks(uint32_t parts) { return parts < (1u << 22) ? parts : 1u << 22; }

// Workgroups of 256 threads of each part of a preparation launch.
struct PrepareBlocks {
  uint32_t pack = 0, bin = 0, clear = 0, compose = 0;
  constexpr uint32_t total() const { return pack + bin + clear + compose; }
  constexpr bool fits() const { return (int64_t)total() * 256 <= kMaxWorkItemsPerLaunch; }
};

// 32-bit words per fixed-bin row of a hard sweep's LDS histogram: the row's
// counters (u32, or two 16-bit ones per word when packed) and a pad that
// makes the row width odd and not 1 modulo 32.  Unpadded rows of a
// power-of-two width would put every cell of one moving bin in one of the
// 32 LDS banks, and the counts of one wave, whose fixed bins differ by
// noise, would queue on that bank; a skew of 3 banks per row spreads them
// over the banks (a plain +1 skew would line up the anti-diagonals).
constexpr int32_t hist_row_words(int32_t bins, bool packed) {
  const int32_t w = (packed ? (bins + 1) / 2 : bins) + 3;
  return (w & 1) ? w : w + 1;
}
constexpr size_t hist_lds_bytes(int32_t bins, bool packed) {
  return (size_t)bins * (size_t)hist_row_words(bins, packed) * 4;
}

// Whether a launch's LDS fits: its dynamic request within the dynamic
// maximum the kernel was configured for, and dynamic plus the kernel's
// static arrays within what one workgroup of the device may hold.  A launch
// past the second limit fails at dispatch (as an invalid allocation that
// the runtime may report only at a later call), so the launchers test it
// before launching.
inline bool lds_fits(size_t dynamic_bytes, size_t static_bytes, size_t configured_dynamic_max,
                     size_t device_max) {
  return dynamic_bytes <= configured_dynamic_max && static_bytes <= device_max &&
         dynamic_bytes <= device_max - static_bytes;
}

// Slabs per transform (a multiple of 8, at least `least` rounded up) of a
// hard sweep of n transforms over `voxels` fixed voxels, with `slots`
// workgroups resident on the device at once.  Workgroups are dealt out as
// slots free up, so a launch takes about `rounds` workgroup times: n c / slots
// and a share of the last workgroup, or as many whole ones as its slots need;
// a workgroup takes its voxels and the clearing and flushing of its LDS
// histogram, worth 4096 + B^2 / 8 voxels; and a transform's slabs add into
// the same few busy cells of one histogram, 8 voxels each.  The constants
// are fitted to sweeps of 64^3 to 256x256x180 volumes, 1 to 200 transforms
// and 32 to 256 bins over 8 to 1024 slabs, where the choice is within a few
// percent of the best.  Against max(2048 / n, 32) slabs, whole calls: 64^3,
// 21 transforms, 32 bins 62 -> 46 us; 128^3, one, 64 bins 68 -> 46 us;
// 256x256x180, one, 128 bins 117 -> 97 us.
inline int64_t planned_slabs(int64_t voxels, int64_t n, int64_t slots, int32_t bins, int64_t least) {
  const double over = 4096.0 + bins * (double)bins / 8.0;
  int64_t best = (least + 7) / 8 * 8;
  if (best < 8) best = 8;
  double least_cost = 1e300;
  for (int64_t c = best; c <= 1024; c += 8) {
    const double r = (double)(n * c) / (double)slots;
    const double whole = (double)((n * c + slots - 1) / slots);
    const double rounds = r + 0.3 > whole ? r + 0.3 : whole;
    const double cost = rounds * ((double)voxels / (double)c + over) + 8.0 * (double)c;
    if (cost < least_cost) {
      least_cost = cost;
      best = c;
    }
  }
  return best;
}

// A transform's share of a thin-slab sweep: `chunks` workgroups (a multiple of
// 8), of which the first `slabs` have a slab each; the slabs divide slab_nz
// slices evenly (the fixed volume's, or a few more: the last are past its end).
struct SlabSplit {
  int32_t chunks, slabs, slab_nz;
};

// Slabs of whole slices, or of even parts of one, keep the workgroups that run
// at once on the same rows of neighbouring slices, whose images share cache
// lines; they matter where the moving layout is far larger than the L2s.
//
// Not turned: planned_slabs' count c, or the least count of aligned slabs within
// 0.7 and 1.1 of it that makes whole rounds (512x512x64 i16, 64 bins, eight
// transforms: 176 slabs 441 us, 192 384; four: 352 307, 256 264).
constexpr int64_t aligned_rounds(int64_t c, int32_t nz, int64_t n, int64_t slots, int64_t least) {
  for (int64_t a = (c * 7 + 9) / 10; a * 10 <= c * 11; ++a)
    if (a % 8 == 0 && a >= least && (a % nz == 0 || nz % a == 0) && n * a % slots == 0) return a;
  return c;
}

// One or two transforms that are turned (the gathers wait longer, and more
// workgroups overlap their waits): even parts of a slice, the count that takes
// the fewest steps of a row group a wave over its whole rounds, the nearest to
// 1.4 workgroups a slot among equals.  Turned by 60 and 90 degrees about y, us a
// call with planned_slabs' count and this: 256x256x180 u16, 128 bins, one
// transform 155 and 215, 125 and 166 (the copy), 180 and 186, 125 and 138 (octs), two
// 245 and 258, 169 and 180; u8, one 146 and 161, 114 and 122.
inline SlabSplit turned_slabs(int32_t ny, int32_t nz, int64_t n, int64_t slots, int32_t waves) {
  const int64_t G = (ny + 3) / 4;
  const double target = 1.4 * (double)slots;
  SlabSplit best{0, 0, 0};
  int64_t least = 0;
  double off = 0.0;
  for (int64_t j = 1; j <= G && j <= 16; ++j) {
    const int64_t slabs = nz * j, per = (G + j - 1) / j;  // row groups of the largest slab
    const int64_t steps = (n * slabs + slots - 1) / slots * ((per + waves - 1) / waves);
    const double ratio = (double)slabs > target ? (double)slabs / target : target / (double)slabs;
    if (best.chunks == 0 || steps < least || (steps == least && ratio < off)) {
      least = steps;
      off = ratio;
      best = SlabSplit{(int32_t)((slabs + 7) / 8 * 8), (int32_t)slabs, nz};
    }
  }
  return best;
}

// ---------------------------------------------------------------------------
// the fixed-volume walk shared by the sweep kernels
// ---------------------------------------------------------------------------

constexpr int kTileX = 16, kTileY = 4;  // a wave64 covers 16 x 4 fixed voxels at a time

// Fixed bins of the hard sweeps.  Each whole run of kFixedRun voxels of a row
// is stored so that the four bytes at 4 dx hold voxels dx, 16 + dx, 32 + dx
// and 48 + dx: the bins a lane needs in four consecutive x steps of 16, in
// one 32-bit load.  The rest of a row (fewer than kFixedRun voxels) stays in
// order.  x of the voxel stored at position p of a row of nx:
constexpr int32_t kFixedRun = 64;
constexpr int32_t fixed_run_x(int32_t p, int32_t nx) {
  if (p >= nx / kFixedRun * kFixedRun) return p;
  const int32_t r = p & (kFixedRun - 1);
  return (p - r) + (r >> 2) + kTileX * (r & 3);
}

// The same for brick sweeps, whose lanes step by 4 along x: in each whole run
// of 16 voxels the four bytes at 4 dx hold voxels dx, 4 + dx, 8 + dx, 12 + dx.
constexpr int32_t kCubeRun = 16;
constexpr int32_t cube_run_x(int32_t p, int32_t nx) {
  if (p >= nx / kCubeRun * kCubeRun) return p;
  const int32_t r = p & (kCubeRun - 1);
  return (p - r) + (r >> 2) + 4 * (r & 3);
}

// Tiled octs of a moving volume: the records of a block of 2 x 2 x 2 voxels
// (16-byte records) or 4 x 2 x 2 (8-byte ones) share a 128-byte line, x
// fastest, then y, z; blocks in x, y, z order, the last ones padded.
constexpr int32_t tile_pad_x(int32_t nx, bool rec8) { return rec8 ? (nx + 3) & ~3 : (nx + 1) & ~1; }
constexpr int32_t tile_pad(int32_t n) { return (n + 1) & ~1; }
constexpr size_t tiled_records(int32_t nx, int32_t ny, int32_t nz, bool rec8) {
  return (size_t)tile_pad_x(nx, rec8) * (size_t)tile_pad(ny) * (size_t)tile_pad(nz);
}
// Record index of voxel (ix, iy, iz), px and py the padded extents:
constexpr uint32_t tiled_index(uint32_t ix, uint32_t iy, uint32_t iz, uint32_t px, uint32_t py, bool rec8) {
  // ((block z * blocks y + block y) * blocks x + block x) * records + place,
  // written as a linear form less what the low bits add too much
  const uint32_t lx = ix & (rec8 ? 3u : 1u), ly = iy & 1u, lz = iz & 1u, s = rec8 ? 4u : 2u;
  return (iz * (py / 2) + iy) * (2 * px) + 4 * ix - 3 * lx - (2 * px - s) * ly - (px * py - 2 * s) * lz;
}

// The rods that brick sweeps cut the fixed volume into: segments of the x axis,
// all `width` voxels but the last, by 16 rows, 2^ly along y and 16 / 2^ly along z
// (one wave step: 4 voxels of each row).
constexpr int32_t kRodX = 64;
struct Rods {
  int32_t width = kRodX, segments = 1, ly = 2;
  constexpr int32_t ry() const { return 1 << ly; }
  constexpr int32_t rz() const { return 16 >> ly; }
  constexpr int32_t last(int32_t nx) const { return nx - (segments - 1) * width; }
  constexpr int32_t longest(int32_t nx) const { return last(nx) > width ? last(nx) : width; }
  constexpr int32_t gy(int32_t ny) const { return (ny + ry() - 1) >> ly; }
  constexpr int32_t gz(int32_t nz) const { return (nz + rz() - 1) >> (4 - ly); }
  constexpr int64_t count(int32_t ny, int32_t nz) const { return (int64_t)segments * gy(ny) * gz(nz); }
};
constexpr Rods cube_rods(int32_t nx) { return Rods{kRodX, (nx + kRodX - 1) / kRodX, 2}; }

// Whether a brick sweep's slabs are dealt to the XCDs in turn, not by eighths of
// the fixed volume (block_work).  The eighths of a volume that is long in x are its
// x segments: turned out of a short axis, those away from the middle lie outside the
// moving volume, and their XCDs idle.  In turn the XCDs fetch more lines twice (us,
// 100 transforms of 0, up to +-20, 0 to 90 and 90 degrees, by eighths and in turn:
// 512x512x200 i16 8874 and 8806, 8237 and 8179, 8548 and 6527, 8878 and 4635;
// 256x256x128 u16 1293 and 1293, 1178 and 1244, 1333 and 1113, 1343 and 856;
// 64x256x256 681 and 685, 555 and 589, 411 and 588, 333 and 661; 128^3 u8, 216 of up
// to 180 degrees, 637 and 651).
constexpr bool deal_slabs(int32_t nx, int32_t ny, int32_t nz) { return nx >= 2 * (ny < nz ? ny : nz); }
// Slab `chunk` by eighths -> the slab dealt in its place; chunks a multiple of 8.
constexpr uint32_t dealt_slab(uint32_t chunk, uint32_t chunks) {
  const uint32_t c8 = chunks >> 3;
  return (chunk % c8) * 8 + chunk / c8;
}

// A slab's walk in brick sweeps: the rods are numbered by
// x segment, then by blocks of yb rods along y, then z, then y within the
// block; a slab is a contiguous range of that numbering, so a block of one
// segment about as high as deep: nearly a cube of the fixed volume, whose image
// stays compact under any rotation.  The waves take a slab's rods in turn, so
// that neighbouring rods are swept at the same time.
struct RodWalk {
  int64_t u, u1;
  int32_t xs, b0, bw, gz, gy;  // x segment, y block and its width, z, y within the block
  int32_t Gy, Gz, yb;
  Rods rods;

  constexpr void init(int32_t fnx, int32_t fny, int32_t fnz, int32_t chunks, uint32_t chunk, int wave) {
    init(cube_rods(fnx), fny, fnz, chunks, chunk, wave);
  }
  constexpr void init(const Rods& r, int32_t fny, int32_t fnz, int32_t chunks, uint32_t chunk, int wave) {
    rods = r;
    Gy = r.gy(fny);
    Gz = r.gz(fnz);
    const int64_t n = r.count(fny, fnz);
    u = n * chunk / chunks;
    u1 = n * (chunk + 1) / chunks;
    const int32_t per = (int32_t)((n + chunks - 1) / chunks);
    yb = 1;
    while (yb < Gy && ((yb * yb) << (2 * r.ly)) < per * 16) ++yb;  // yb ry < per / yb rz
    const int32_t plane = Gy * Gz;  // <= 2^24
    xs = (int32_t)(u / plane);
    const int32_t rem = (int32_t)(u - (int64_t)xs * plane);
    b0 = rem / (yb * Gz) * yb;
    bw = Gy - b0 < yb ? Gy - b0 : yb;
    gz = (rem - b0 * Gz) / bw;
    gy = rem - b0 * Gz - gz * bw;
    next(wave);
  }

  constexpr void next(int32_t n) {
    u += n;
    gy += n;
    while (gy >= bw) {
      gy -= bw;
      if (++gz == Gz) {
        gz = 0;
        b0 += bw;
        if (b0 == Gy) {
          b0 = 0;
          ++xs;
        }
        // the rods left over keep their place in the next block's numbering
        bw = Gy - b0 < yb ? Gy - b0 : yb;
      }
    }
  }
  constexpr int32_t x0() const { return xs * rods.width; }
  constexpr int32_t j0() const { return (b0 + gy) << rods.ly; }
  constexpr int32_t k0() const { return gz << (4 - rods.ly); }
};

// The rods of a fixed volume.  Segments: about 64 voxels and nearly equal (48 to
// 96), so that slabs, which are ranges of rods, hold nearly equal work (80x96x96
// in segments of 64 and 16: 408 us for 216 transforms, of 80: 288).  Rows: the
// cross-section that leaves the fewest lanes without a voxel, the flatter ones
// weighted by what they cost where none is left over: the nearer to 4 x 4, the
// fewer cache lines a wave's image touches.  In a fixed volume of at most 8
// slices (or rows) the flat ones win by themselves: a turned one lies mostly
// outside, and their rods are outside as a whole more often (nz = 8: 160, 149,
// 148 in the terms below).  8 pairs of 256x256xnz u8, 16
// transforms each, 32 bins, us a call with 4x4, 8x2 and 16x1 rows: nz = 5 138,
// 120, 110; 9 192, 169, 159; 17 281, 264, 271; 3 of nz = 64 363, 373, 400; 216
// rotations of up to 180 degrees, 256x256x180 u16: 5428, 5820, 6809.
inline Rods rods_for(int32_t nx, int32_t ny, int32_t nz) {
  Rods r;
  r.segments = nx < 96 ? 1 : (nx + 31) / 64;
  r.width = (nx + 8 * r.segments) / (16 * r.segments) * 16;
  if (r.width < 16) r.width = 16;
  constexpr double weight[5] = {1.15, 1.05, 1.0, 1.05, 1.15};
  double least = 1e300;
  for (int32_t ly : {2, 3, 1, 4, 0}) {
    const Rods c{r.width, 1, ly};
    const bool thin = (ly > 2 && nz <= 8) || (ly < 2 && ny <= 8);
    const double cost = (thin ? 0.9 : 1.0) * weight[ly] * (double)c.count(ny, nz);
    if (cost < least) {
      least = cost;
      r.ly = ly;
    }
  }
  return r;
}

// Lanes per row group of the pass that turns fixed bins into slots: a lane per
// wave tile, rounded up to a power of two, so that a wave of 64 takes 64 / span
// row groups and few of its lanes idle (whole Parzen calls on one transform
// without overlap, us, a wave per row group and this: 2x512x512 137 and 44,
// 16x256x256 62 and 43, 128^3 49 and 47, 256x256x180 77 and 66, 512x512x300 190
// and 169).
constexpr int32_t slots_span(int32_t nx) {
  int32_t span = 1;
  while (span < 64 && span * kTileX < nx) span *= 2;
  return span;
}

// One wave's walk over its share of a slab: groups of kTileY consecutive
// rows of one slice with exact Q32 row coordinates.  Either each wave takes
// a contiguous share of the slab's row groups (GroupWalk), or the waves
// take them in turn (wave w: groups w, w + NW, ...; GroupWalkFlex with
// `interleave`, chosen at run time).  Where the
// work per row group is even (a hard sweep; the background band of a Parzen
// sweep) contiguous shares keep each wave on neighbouring rows; where it is
// concentrated in a few rows (a Parzen band of rare slots, the skull of a
// CT), contiguous shares leave most waves idle while the few that hold those
// rows finish, and interleaving spreads them over all waves.
// Lane (dx, dy) of the 16 x 4 tile starts at r + lane_off and steps by
// `step` = 16 M[:,0] along x.
// (Constexpr members, so the same code runs in the kernels and in the CPU
// test of the walk.)
template <bool FLEX>
struct GroupWalkT {
  int64_t g, g1;
  int32_t j0, k, G, stride;
  int64_t r[3], lane_off[3], step[3], adv[3], wrap[3];

  constexpr void init(const int64_t* Mq, int32_t fny, int32_t fnz, int32_t chunks, uint32_t chunk, int wave,
                      int nwaves, int dx, int dy, bool interleave = false, int32_t slab_nz = 0) {
    G = (fny + kTileY - 1) / kTileY;
    // slab_nz: slices that the slabs divide evenly, at least fnz (0: fnz)
    const int64_t groups = (int64_t)G * fnz, even = slab_nz ? (int64_t)G * slab_nz : groups;
    const int64_t e0 = even * chunk / chunks, e1 = even * (chunk + 1) / chunks;
    const int64_t s0 = e0 < groups ? e0 : groups, s1 = e1 < groups ? e1 : groups;
    if (FLEX && interleave) {
      g = s0 + wave;
      g1 = s1;
      stride = nwaves;
    } else {
      g = s0 + (s1 - s0) * wave / nwaves;
      g1 = s0 + (s1 - s0) * (wave + 1) / nwaves;
      stride = 1;
    }
    k = (int32_t)(g / G);
    j0 = (int32_t)(g - (int64_t)k * G) * kTileY;
    for (int a = 0; a < 3; ++a) {
      const int64_t m0 = Mq[4 * a], m1 = Mq[4 * a + 1], m2 = Mq[4 * a + 2], m3 = Mq[4 * a + 3];
      r[a] = m1 * j0 + m2 * k + m3;
      lane_off[a] = m0 * dx + m1 * dy;
      step[a] = m0 * kTileX;
      adv[a] = m1 * (FLEX ? (int64_t)kTileY * stride : (int64_t)kTileY);
      wrap[a] = m2 - m1 * ((int64_t)G * kTileY);
    }
  }

  constexpr void next() {
    const int32_t st = FLEX ? stride : 1;
    g += st;
    j0 += st * kTileY;
    for (int a = 0; a < 3; ++a) r[a] += adv[a];
    if constexpr (FLEX) {
      while (j0 >= G * kTileY) {  // into the next slice (more than once when a slice has fewer groups than waves)
        j0 -= G * kTileY;
        ++k;
        for (int a = 0; a < 3; ++a) r[a] += wrap[a];
      }
    } else if (j0 >= G * kTileY) {
      j0 = 0;
      ++k;
      for (int a = 0; a < 3; ++a) r[a] += wrap[a];
    }
  }
};
using GroupWalk = GroupWalkT<false>;
using GroupWalkFlex = GroupWalkT<true>;

// ---------------------------------------------------------------------------
// x ranges of a row group: where every lane of the tile lies inside the
// moving volume, and where some lane can
// ---------------------------------------------------------------------------
//
// Along a row group the 64 lanes of the tile step together by
// step_a = 16 m0_a per x iteration, so at iteration `it` the least and the
// greatest coordinate over the tile on axis a are R_a + omin_a + it step_a
// and R_a + omax_a + it step_a, where R_a = m1_a j0 + m2_a k + m3_a is the
// coordinate of the group's first voxel and omin_a, omax_a are the extreme
// lane offsets m0_a dx + m1_a dy.  Every lane lies in [0, top_a] on every
// axis exactly when six inequalities A + it S >= 0 hold: A = R + omin with
// S = step, and A = top - R - omax with S = -step, for each axis.  Some lane
// can lie inside only when the six with omin and omax exchanged hold.  One
// with S > 0 bounds `it` from below (it >= ceil(-A / S)), one with S < 0
// from above (it <= floor(A / -S)), and one with S = 0 holds for every `it`
// or for none.
//
// Sixteen lanes evaluate the twelve bounds of a row group at once.  Lane l
// takes axis l % 4 (none when 3) of group l / 4: lower bounds of the
// every-lane range, its upper bounds, lower bounds of the some-lane range,
// its upper bounds.  It forms v = floor((A + D) / |S|), which is the upper
// bound itself, or minus the lower bound, so that each group's bound is the
// least v of its four lanes.  The margin D = -/+ (ceil(|S| / 64) + 1) (every-
// lane / some-lane range) is an integer of at least |S| / 64, so A + D stays
// an exact integer in double (below 2^53), and the division and the
// rounding to float err by far less than D / |S|: the every-lane range can
// only come out narrower than exact, the some-lane range only wider, by one
// iteration where a bound lies within D / |S| of an integer (a face hit
// exactly is one such case).  When a transform's entries are too large for
// A to be exact the lane says so (`exact` false) and the caller checks
// every voxel.

// range_lane and range_value use math builtins and so cannot be constexpr;
// compiled as HIP they are marked for both sides.
#ifdef __HIP__
#define GEMI_HOST_DEVICE __attribute__((host, device))
#else
#define GEMI_HOST_DEVICE
#endif

struct RangeLane {
  double a1, a2, a0;  // A + D = a1 j0 + a2 k + a0
  double inv;         // v = floor((A + D) inv)
  bool exact;
};

constexpr float kRangeClamp = 1048576.0f;  // |v| <= 2^20, far past any row's iterations

// The constants of lane `lane` (0..63), given the Q32 entries (m0, m1, m2,
// m3) of the matrix row of its axis (lane % 4; any values for the lanes that
// take no bound) and that axis's upper moving coordinate top = (n - 1) 2^32,
// all as doubles (integers; exact below 2^53).  Everything is formed in
// double: while |m0| < 2^47, |m1|, |m2| < 2^38 and |m3| < 2^49 (`exact`)
// every value below is an integer below 2^53 (a half-integer below 2^51
// when S = 0, which makes m0 = 0) and so exact.
GEMI_HOST_DEVICE inline RangeLane range_lane(int lane, double m0, double m1, double m2, double m3, double top) {
  RangeLane c{0.0, 0.0, 1073741824.0, 1.0, true};  // no bound: v clamps to 2^20
  if (lane >= 16 || (lane & 3) == 3) return c;
  const int group = lane >> 2;
  const bool every = group < 2, lower = (group & 1) == 0;
  const double step = m0 * kTileX;
  const double ox = m0 * (kTileX - 1), oy = m1 * (kTileY - 1);
  const double omin = (ox < 0 ? ox : 0.0) + (oy < 0 ? oy : 0.0);
  const double omax = (ox > 0 ? ox : 0.0) + (oy > 0 ? oy : 0.0);
  // "lo": R + o_lo + it step >= 0; "hi": top - R - o_hi - it step >= 0
  const double o_lo = every ? omin : omax, o_hi = every ? omax : omin;
  const bool lo = lower == (step >= 0);
  const double mag = __builtin_fabs(step);
  const double margin = __builtin_floor(mag * (1.0 / 64.0)) + 2.0;  // ceil(|S| / 64) + 1 at least
  const double cst = lo ? m3 + o_lo : top - o_hi - m3;
  c.a1 = lo ? m1 : -m1;
  c.a2 = lo ? m2 : -m2;
  // S = 0: v is +-2^20 by the sign of A + 1/2 (no margin: A is an integer)
  c.a0 = step == 0 ? cst + 0.5 : cst + (every ? -margin : margin);
  c.inv = step == 0 ? 1152921504606846976.0 : 1.0 / mag;  // 2^60 when S = 0
  // j0, k < 2^12: |A + D| < 2^50 + 2^50 + |m3| + 15 |m0| + 3 |m1| + top + margin < 2^53
  c.exact = __builtin_fabs(m0) < 140737488355328.0 && __builtin_fabs(m1) < 274877906944.0 &&
            __builtin_fabs(m2) < 274877906944.0 && __builtin_fabs(m3) < 562949953421312.0;
  return c;
}

// v of one lane for the row group whose first row is j0 in slice k.
GEMI_HOST_DEVICE inline int32_t range_value(const RangeLane& c, int32_t j0, int32_t k) {
  const double A = __builtin_fma((double)j0, c.a1, __builtin_fma((double)k, c.a2, c.a0));
  const float t = __builtin_fminf(__builtin_fmaxf((float)(A * c.inv), -kRangeClamp), kRangeClamp);
  return (int32_t)__builtin_floorf(t);
}

// Iterations of a row group of `full` x steps: checked [u0, c0), every lane
// inside [c0, c1), checked [c1, u1); none left out when `skip` is false
// (CLAMP counts every voxel).  The arguments are the least v of the four
// groups of lanes.
struct RowSpans {
  int32_t u0, c0, c1, u1;
};
constexpr RowSpans row_spans(int32_t v_every_lo, int32_t v_every_hi, int32_t v_some_lo, int32_t v_some_hi,
                             int32_t full, bool skip) {
  RowSpans s{0, 0, 0, full};
  if (skip) {
    s.u0 = -v_some_lo > 0 ? (-v_some_lo < full ? -v_some_lo : full) : 0;
    s.u1 = v_some_hi + 1 < full ? v_some_hi + 1 : full;
    if (s.u1 < s.u0) s.u1 = s.u0;
  }
  s.c0 = -v_every_lo > s.u0 ? -v_every_lo : s.u0;
  s.c1 = v_every_hi + 1 < s.u1 ? v_every_hi + 1 : s.u1;
  if (s.c1 <= s.c0) s.c0 = s.c1 = s.u1;
  return s;
}

// Sampled Parzen calls: the rise from which the moving volume is laid out in
// records (launch_sample_layout).
// The copy's gain is that a line holds several samples of a row; turned, each
// sample has lines of its own, four of the copy against one of the octs or two
// of the quads, and sparse samples (3% and less) share none even upright.
// With a 16-bit copy of mb MB (of the same dims, for a float volume), the records save a transform samples * k (sqrt(rise) - c),
// in us and millions, and cost P us more to write; fitted to 15 volumes of 64^3
// to 320x320x200 (u8, u16, i16, f32), fractions of 1 to 30%, 20 and 100 rotations
// of ten families: the choice is within 0.5% of the better layout over all of
// them, and no call is more than 3% over what it took when the records were the
// only layout (us, copy and records, 100 rotations:
// 256x256x180 u16 up to +-10 degrees about y, 3% 644 and 436, 10% 1327 and 1115; up
// to +-3, 10% 736 and 840; 192^3 f32, 10%, +-10 1212 and 1590, +-90 2310 and 1953).
inline double sample_layout_limit(double samples, double fraction, size_t copy_bytes, double n, bool f32) {
  auto least = [](double a, double b) { return a < b ? a : b; };
  const double mb = (double)copy_bytes * 1e-6;
  const double c = f32 ? least(0.5, 0.55 - 0.013 / fraction) : least(least(0.27, 0.12 + 0.006 * mb), 0.33 - 0.015 / fraction);
  const double P = f32 ? 5.0 + mb * least(0.07 * mb, 4.5) : 18.0 + mb * least(0.05 * mb, 4.0);
  const double root = (c > 0.0 ? c : 0.0) + P / (n * samples * 1e-6 * (f32 ? 4.5 : 5.5) * sqrt(mb));
  return root * root;
}
// A row further in the slice is nearer than one in the next slice: where samples
// are sparse, on the same page (256x256x180 u16, rise of 0.08 from M[1][0] and from
// M[2][0], records' gain: 1% of the voxels 4 and 28%, 10% 26 and 19%, 30% 17 and 2%).
inline double sample_row_weight(double fraction) {
  const double w = 0.1 + 2.5 * fraction;
  return w < 0.85 ? w : 0.85;
}

}  // namespace gemi
