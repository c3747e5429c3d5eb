"""CPU test of the preparation launch's workgroup counts (csrc/plan.h),
compiled with g++: a dispatch counts its work-items in 32 bits, and rows of
few voxels give up to 2^24 row parts, so those are taken in turns.  At the
largest of every part (octs of the flattest moving volumes, fixed volumes
and tables of any size, 2^24 transforms) the launch stays below 2^31
work-items, and every row part is some workgroup's."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1909_10690_amd", "csrc")

PROGRAM = r"""
#include "plan.h"
#include <stdio.h>
using namespace gemi;
int main() {
  int bad = 0;
  const int dims[][3] = {{2, 2, 2},        {2, 4096, 4096},  {15, 4096, 4096},  {16, 4096, 4095}, {16, 4096, 4096},
                         {16, 4093, 4091}, {64, 2048, 2048}, {256, 1024, 1024}, {257, 1021, 1021}, {4096, 256, 256},
                         {256, 256, 180}};
  for (const auto& d : dims) {
    const uint32_t parts = row_parts(d[0], d[1], d[2]);
    if (parts != (uint64_t)((d[0] + 255) / 256) * d[1] * d[2]) { printf("parts %u\n", parts); ++bad; }
    PrepareBlocks nb;
    nb.pack = row_part_blocks(parts);
    nb.bin = nb.clear = fill_blocks((size_t)-1 / 2);
    nb.compose = 4096;
    if (!nb.fits() || nb.total() * 256ull > 0x7FFFFFFFull) { printf("%d %d %d: %u\n", d[0], d[1], d[2], nb.total()); ++bad; }
    if (nb.pack < 1 || nb.pack > parts) { printf("blocks %u\n", nb.pack); ++bad; }
    // the parts a workgroup takes, block + k nb < 2^32, cover [0, parts)
    uint64_t covered = 0;
    for (uint32_t b = 0; b < nb.pack; ++b) covered += (parts - 1 - b) / nb.pack + 1;
    if (covered != parts || (uint64_t)parts + nb.pack > 0xFFFFFFFFull) { printf("covered %llu\n", (unsigned long long)covered); ++bad; }
    // clinical volumes keep a workgroup per row part
    if (parts <= (1u << 22) && nb.pack != parts) ++bad;
  }
  if (fill_blocks(0) != 1 || fill_blocks(256) != 1 || fill_blocks(257) != 2 || fill_blocks(1 << 28) != 8192) ++bad;
  PrepareBlocks wrapped;
  wrapped.pack = 1u << 24;
  if (wrapped.fits()) { printf("2^24 workgroups accepted\n"); ++bad; }
  printf(bad ? "FAIL %d\n" : "OK\n", bad);
  return bad != 0;
}
"""


def test_prepare_blocks(tmp_path):
    src, exe = tmp_path / "p.cpp", tmp_path / "p"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", str(exe), str(src)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip().endswith("OK"), out.stdout + out.stderr


def test_launcher_uses_the_counts():
    """The launcher takes its counts from these functions and refuses a grid that would wrap."""
    text = open(os.path.join(CSRC, "hard.hip")).read()
    assert "row_part_blocks(row_parts(" in text and "nb.fits()" in text
