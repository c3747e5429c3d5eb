"""CPU tests of the hard sweeps' stored bin order, brick walk,
tiled records and slab count (csrc/plan.h),
compiled with g++: a multiple of 8 in range, never below the L2 bound, and
above it never so many that a workgroup's voxels are few beside its table."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1909_10690_amd", "csrc")

PROGRAM = r"""
#include "plan.h"
#include <initializer_list>
#include <stdio.h>
using namespace gemi;
int main() {
  int bad = 0;
  const long long voxels[] = {8, 4096, 110592, 262144, 2097152, 11796480, 268435456};
  const long long ns[] = {1, 2, 21, 512, 1000, 1 << 24};
  const long long least[] = {0, 1, 32, 120, 2731};
  for (long long v : voxels)
    for (long long n : ns)
      for (long long slots : {256LL, 512LL, 2048LL})
        for (int bins : {2, 32, 128, 256})
          for (long long l : least) {
            const long long c = planned_slabs(v, n, slots, bins, l);
            const long long low = l < 8 ? 8 : (l + 7) / 8 * 8;
            if (c % 8 || c < low || (c > 1024 && c != low)) { printf("c=%lld v=%lld n=%lld l=%lld\n", c, v, n, l); ++bad; }
            if (c > low && v / c < 100) { printf("c=%lld v=%lld n=%lld: too many\n", c, v, n); ++bad; }
          }
  // one transform of a clinical volume fills most of the slots in one round
  const long long c = planned_slabs(11796480, 1, 512, 128, 16);
  if (c < 256 || c > 512) { printf("single: %lld\n", c); ++bad; }
  printf(bad ? "FAIL %d\n" : "OK\n", bad);
  return bad != 0;
}
"""


RUNS = r"""
#include "plan.h"
#include <initializer_list>
#include <stdio.h>
#include <vector>
using namespace gemi;
int main() {
  int bad = 0;
  for (int nx = 2; nx <= 300; ++nx) {
    std::vector<int> seen(nx, 0);
    for (int p = 0; p < nx; ++p) {
      const int x = fixed_run_x(p, nx);
      if (x < 0 || x >= nx) { ++bad; continue; }
      ++seen[x];
    }
    for (int x = 0; x < nx; ++x) bad += seen[x] != 1;
    // step it of lane dx of a whole run: byte it % 4 of the word at 4 dx
    for (int it = 0; it < nx / kFixedRun * 4; ++it)
      for (int dx = 0; dx < kTileX; ++dx)
        bad += fixed_run_x((it >> 2) * kFixedRun + 4 * dx + (it & 3), nx) != it * kTileX + dx;
  }
  printf(bad ? "FAIL %d\n" : "OK\n", bad);
  return bad != 0;
}
"""


def test_fixed_runs(tmp_path):
    """The stored order of the fixed bins is a permutation of each row, and
    holds the bins where the sweep reads them."""
    src, exe = tmp_path / "r.cpp", tmp_path / "r"
    src.write_text(RUNS)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", str(exe), str(src)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr


BRICKS = r"""
#include "plan.h"
#include <initializer_list>
#include <stdio.h>
#include <vector>
using namespace gemi;
int main() {
  int bad = 0;
  for (int nx = 2; nx <= 70; ++nx) {
    std::vector<int> seen(nx, 0);
    for (int p = 0; p < nx; ++p) ++seen[cube_run_x(p, nx)];
    for (int x = 0; x < nx; ++x) bad += seen[x] != 1;
    for (int x = 0; x < nx / kCubeRun * kCubeRun; ++x)  // step x / 4 of lane x % 4
      bad += cube_run_x((x & ~15) + 4 * (x & 3) + ((x >> 2) & 3), nx) != x;
  }
  // every rod once over the slabs and waves
  for (int nx : {2, 64, 65, 200})
    for (int ny : {2, 4, 5, 33, 64})
      for (int nz : {2, 7, 48})
        for (int chunks : {8, 24, 120, 1024})
          for (int nw : {4, 8, 16}) {
            const int X = (nx + 63) / 64, Y = (ny + 3) / 4, Z = (nz + 3) / 4;
            std::vector<int> seen((size_t)X * Y * Z, 0);
            for (int c = 0; c < chunks; ++c)
              for (int w = 0; w < nw; ++w) {
                RodWalk k{};
                k.init(nx, ny, nz, chunks, c, w);
                for (; k.u < k.u1; k.next(nw)) {
                  const int x = k.x0() / 64, y = k.j0() / 4, z = k.k0() / 4;
                  if (x < 0 || x >= X || y < 0 || y >= Y || z < 0 || z >= Z) { ++bad; break; }
                  ++seen[((size_t)x * Y + y) * Z + z];
                }
              }
            for (int v : seen) bad += v != 1;
          }
  // tiled records: all different, and each block's records one 128-byte line
  for (int r8 = 0; r8 < 2; ++r8)
    for (int nx : {2, 3, 4, 8, 37})
      for (int ny : {2, 3, 10})
        for (int nz : {2, 5, 14}) {
          const int w = r8 ? 4 : 2, px = tile_pad_x(nx, r8), py = tile_pad(ny);
          bad += px % w || py % 2 || px < nx || py < ny || tiled_records(nx, ny, nz, r8) % (4 * w);
          std::vector<int> seen(tiled_records(nx, ny, nz, r8), 0);
          for (int z = 0; z < nz; ++z)
            for (int y = 0; y < ny; ++y)
              for (int x = 0; x < nx; ++x) {
                const uint32_t i = tiled_index(x, y, z, px, py, r8);
                if (i >= seen.size()) { ++bad; continue; }
                bad += seen[i]++;
                const uint32_t block = ((z / 2) * (py / 2) + y / 2) * (px / w) + x / w;
                bad += i != block * 4 * w + (z % 2) * 2 * w + (y % 2) * w + x % w;
              }
        }
  printf(bad ? "FAIL %d\n" : "OK\n", bad);
  return bad != 0;
}
"""


def test_bricks(tmp_path):
    """The brick sweeps' walk visits every rod once; the stored bins and the
    tiled records are permutations with the places the sweep computes."""
    src, exe = tmp_path / "b.cpp", tmp_path / "b"
    src.write_text(BRICKS)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", str(exe), str(src)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr


def test_planned_slabs(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", str(exe), str(src)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
