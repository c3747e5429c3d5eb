"""Layout of a sampled Parzen call's moving volume (sample_layout_limit and
sample_row_weight, csrc/plan.h, compiled with g++) against measured calls on both
sides of the limit: us with the plain copy and with records, n rotations."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1909_10690_amd", "csrc")

PROGRAM = r"""
#include "plan.h"
#include <stdio.h>
using namespace gemi;
struct Call { int x, y, z; bool f32; double fraction; int n; double row, slice, copy, records; };
int main() {
  const Call calls[] = {
      {256, 256, 180, false, 0.03, 100, 0.0, 0.079, 643.9, 436.2}, {256, 256, 180, false, 0.03, 100, 0.0, 0.024, 441.6, 358.6},
      {256, 256, 180, false, 0.03, 20, 0.0, 0.029, 189.2, 203.0},  {256, 256, 180, false, 0.1, 100, 0.0, 0.079, 1327.1, 1114.9},
      {256, 256, 180, false, 0.1, 100, 0.0, 0.024, 736.1, 840.4},  {256, 256, 180, false, 0.3, 100, 0.0, 0.048, 1772.1, 1932.4},
      {256, 256, 180, false, 0.3, 100, 0.157, 0.0, 2120.9, 1812.1}, {192, 192, 192, false, 0.03, 100, 0.0, 0.079, 390.3, 272.7},
      {192, 192, 192, false, 0.3, 100, 0.157, 0.0, 1016.0, 850.4}, {192, 192, 192, true, 0.03, 100, 0.0, 0.118, 518.2, 476.2},
      {192, 192, 192, true, 0.1, 100, 0.0, 0.079, 899.4, 1187.9},  {192, 192, 192, true, 0.1, 100, 0.0, 0.339, 1827.3, 1766.6},
      {320, 320, 200, false, 0.3, 100, 0.0, 0.048, 3485.9, 4177.4}, {320, 320, 200, false, 0.1, 100, 0.157, 0.0, 2022.8, 1592.5},
      {128, 128, 128, false, 0.3, 100, 0.0, 0.118, 365.3, 318.5},  {128, 128, 128, false, 0.1, 100, 0.0, 0.048, 177.1, 181.4},
      {64, 64, 64, false, 0.3, 100, 0.0, 1.0, 138.3, 110.5},       {64, 64, 64, false, 0.1, 100, 0.0, 0.339, 72.1, 83.8}};
  int bad = 0;
  for (const Call& c : calls) {
    const double voxels = (double)c.x * c.y * c.z;
    const double limit = sample_layout_limit(c.fraction * voxels, c.fraction, (size_t)(2 * voxels), c.n, c.f32);
    const double rise = sample_row_weight(c.fraction) * c.row + c.slice;
    if ((rise > limit) != (c.records < c.copy)) { printf("%dx%dx%d %d %g n %d: rise %g limit %g\n", c.x, c.y, c.z, c.f32, c.fraction, c.n, rise, limit); ++bad; }
  }
  for (bool f32 : {false, true})  // finite and above 0 at every size
    for (double f : {1e-9, 0.01, 1.0, 3.0})
      for (size_t bytes : {(size_t)32, (size_t)1 << 20, (size_t)1 << 32}) {
        const double limit = sample_layout_limit(1.0, f, bytes, 1, f32);
        if (!(limit > 0.0 && limit < 1e300)) ++bad;
      }
  printf(bad ? "FAIL %d\n" : "OK\n", bad);
  return bad != 0;
}
"""


def test_sample_layout_host(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", str(exe), str(src)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
