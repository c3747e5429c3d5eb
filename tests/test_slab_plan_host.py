"""CPU test of the hard sweeps' slab count (csrc/plan.h, planned_slabs),
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


def test_planned_slabs(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", str(exe), str(src)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
