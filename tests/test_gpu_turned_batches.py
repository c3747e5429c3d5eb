"""Hard calls of few transforms: the slab counts for transforms that are turned
and not (a CPU test of csrc/plan.h, compiled with g++, with the walk that uses
them), and GPU parity on both sides of what the device chooses -- the plain copy
or octs, either count -- against the CPU oracle, histograms bit-exact."""
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_1909_10690_amd import inputs
from paper_1909_10690_amd import transforms as T

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1909_10690_amd", "csrc")

PROGRAM = r"""
#include "plan.h"
#include <initializer_list>
#include <stdio.h>
#include <vector>
using namespace gemi;
int main() {
  const int64_t M[12] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12};
  int bad = 0;
  const int dims[][2] = {{2, 300}, {64, 64}, {5, 181}, {256, 180}, {217, 181}, {512, 64}, {200, 50}, {4, 300}, {300, 9}, {4096, 2}, {2, 8}};
  for (const auto& d : dims)
    for (int n = 1; n <= 8; ++n)
      for (int slots : {256, 512, 2048})
        for (int waves : {4, 8, 16})
          {
            const long long groups = (long long)((d[0] + 3) / 4) * d[1];
            const SlabSplit s = turned_slabs(d[0], d[1], n, slots, waves);
            if (s.chunks % 8 || s.slabs < 1 || s.slabs > s.chunks || s.chunks - s.slabs > 7 || s.slab_nz != d[1]) {
              printf("%d %d n %d: %d %d %d\n", d[0], d[1], n, s.chunks, s.slabs, s.slab_nz); ++bad; continue;
            }
            std::vector<unsigned char> seen(groups, 0);  // the walk: every row group once
            for (int c = 0; c < s.chunks; ++c)
              for (int w = 0; w < waves; ++w) {
                GroupWalk k;
                k.init(M, d[0], d[1], s.slabs, c, w, waves, 0, 0, false, s.slab_nz);
                for (; k.g < k.g1; k.next()) {
                  if (k.g < 0 || k.g >= groups || c >= s.slabs) { ++bad; break; }
                  ++seen[k.g];
                }
              }
            for (unsigned char v : seen) bad += v != 1;
          }
  for (int c : {8, 24, 112, 176, 352, 360, 1024})
    for (int nz : {2, 64, 128, 180, 181})
      for (int n : {1, 4, 8, 1000}) {
        const long long a = aligned_rounds(c, nz, n, 512, 40);
        if (a % 8 || (a != c && (a < 40 || a * 10 < c * 7 || a * 10 > c * 11 || n * a % 512))) { printf("c %d nz %d n %d: %lld\n", c, nz, n, a); ++bad; }
      }
  if (aligned_rounds(176, 64, 8, 512, 171) != 192 || aligned_rounds(352, 64, 4, 512, 171) != 256) ++bad;
  printf(bad ? "FAIL %d\n" : "OK\n", bad);
  return bad != 0;
}
"""


def test_slab_splits_host(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", str(exe), str(src)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr


def rotation(deg, centre, shift=(0, 0, 0)):
    return T.centred_matrix(T.affine_matrix(deg), shift, centre)


@pytest.mark.gpu
@pytest.mark.parametrize("mdt,hi", [(np.uint8, 255), (np.uint16, 4095), (np.uint16, 65535), (np.int16, 700)])
@pytest.mark.parametrize("clamp", [0, 1])
@pytest.mark.parametrize("ms", [(100, 91, 83), (180, 160, 150)])
def test_both_sides_of_the_choices(mdt, hi, clamp, ms):
    """The smaller moving volume has the layout chosen, for up to four
    transforms; the larger one, in 16 bits, the slab count."""
    import torch
    from paper_1909_10690_amd import binding as B
    rng = np.random.default_rng(hi + clamp)
    fs = (128, 120, 110)
    f, m = inputs.random_volume(rng, fs, np.uint8, 0, 255), inputs.random_volume(rng, ms, mdt, 0, hi)
    spacing = tuple(a / b for a, b in zip(fs, ms))
    oF = oracle.volume(f, 0, 255)
    oM = oracle.volume(m, 0, hi, spacing=spacing)
    ctx = B.Context(0)
    F, M = B.Volume.from_numpy(f, 0, 255), B.Volume.from_numpy(m, 0, hi, spacing=spacing)
    c = T.fixed_centre(fs)
    shifts = [rotation((0, 0, 0), c, (0.5 * k, -0.25, 0.75)) for k in range(8)]
    turned = [rotation((3 * k, 88 - 4 * k, 2), c, (0.25, 0.5, -k)) for k in range(8)]
    bad = np.full((3, 4), np.nan)
    ws = torch.zeros(ctx.workspace_size(F, M, 8, 64, 1), dtype=torch.uint8, device="cuda")
    layouts, counts = set(), set()
    for mats in (shifts[:1], turned[:1], turned[:2], shifts[:4], turned[:4], turned[:3] + [bad], shifts[:5], turned[:7], turned, shifts[:4] + turned[:4]):
        P = np.stack(mats).reshape(-1, 12)
        for bins in (64, 200):
            print(f"turned {np.dtype(mdt).name} {hi} clamp={clamp} n={len(P)} bins={bins}", flush=True)
            _, oov, oh = oracle.eval_hard(oF, oM, P, bins, (1.0,), boundary=clamp, want_hist=True)
            _, ov, h = ctx.eval(F, M, torch.from_numpy(P).cuda(), bins, (1.0,), flags=clamp, want_hist=True, workspace=ws if bins == 64 else None)
            torch.cuda.synchronize()
            assert np.array_equal(ov.cpu().numpy(), oov)
            assert np.array_equal(h.cpu().numpy().astype(np.uint32), oh)
            if bins == 64:  # what the device chose lies behind the matrices
                at = (96 * len(P) + 255) // 256 * 256
                octs, turn = ws[at:at + 8].cpu().numpy().view(np.uint32)
                if ms[0] == 100 and len(P) == 4:
                    layouts.add(int(octs))
                if ms[0] == 180 and mdt != np.uint8 and len(P) <= 2:
                    counts.add(int(turn))
    assert counts == ({0, 1} if ms[0] == 180 and mdt != np.uint8 else set())
    if clamp and ms[0] == 100:  # every voxel counts: the turned batches of four take octs
        assert layouts == {0, 1}
    ctx.close()
