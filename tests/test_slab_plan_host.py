"""CPU tests of the hard sweeps' stored bin order and slab count (csrc/plan.h),
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


def test_planned_slabs(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", str(exe), str(src)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
