"""The rods of brick sweeps on thin, narrow and ragged fixed volumes: a CPU test
of their cut and walk (csrc/plan.h, compiled with g++) and GPU parity of
bricks and pairs against the CPU oracle, histograms bit-exact."""
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_1909_10690_amd import inputs

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1909_10690_amd", "csrc")

PROGRAM = r"""
#include "plan.h"
#include <initializer_list>
#include <stdio.h>
#include <vector>
using namespace gemi;
int main() {
  int bad = 0;
  for (int nx = 2; nx <= 4096; ++nx) {  // segments: whole runs, none empty, nearly equal
    const Rods r = rods_for(nx, 64, 64);
    if (r.width % kCubeRun || r.last(nx) < 1 || r.longest(nx) > 96 || r.ly != 2) ++bad;
    if (nx >= 32 && nx < 400 && r.longest(nx) * r.segments > nx + nx / 2) { printf("nx %d: %d of %d, %d\n", nx, r.segments, r.width, r.last(nx)); ++bad; }
    if (65535 / (16 * r.longest(nx)) < 1) ++bad;
  }
  // every voxel once over the slabs and waves, whatever the cross-section
  for (int nx : {2, 17, 64, 65, 95, 96, 97, 130})
    for (int ny : {2, 3, 5, 8, 9, 33, 64})
      for (int nz : {2, 5, 7, 8, 13, 48}) {
        const Rods r = rods_for(nx, ny, nz);
        if (r.ry() * r.rz() != 16) ++bad;
        for (int chunks : {8, 24, 1024})
          for (int nw : {8, 16}) {
            std::vector<unsigned char> seen((size_t)nx * ny * nz, 0);
            for (int c = 0; c < chunks; ++c)
              for (int w = 0; w < nw; ++w) {
                RodWalk k{};
                k.init(r, ny, nz, chunks, c, w);
                for (; k.u < k.u1; k.next(nw)) {
                  const int width = k.xs == r.segments - 1 ? nx - k.x0() : r.width;
                  if (k.x0() < 0 || k.x0() + width > nx) { ++bad; break; }
                  for (int z = k.k0(); z < k.k0() + r.rz() && z < nz; ++z)
                    for (int y = k.j0(); y < k.j0() + r.ry() && y < ny; ++y)
                      for (int x = k.x0(); x < k.x0() + width; ++x) ++seen[((size_t)z * ny + y) * nx + x];
                }
              }
            for (unsigned char v : seen) bad += v != 1;
          }
      }
  // flat volumes leave few lanes without a voxel
  for (int n : {2, 3, 5, 6, 7, 8, 9, 17}) {
    const Rods z = rods_for(256, 256, n), y = rods_for(256, n, 256);
    if (z.count(256, n) * z.width * 16 > 256 * 256 * n * 1.2 || y.count(n, 256) * y.width * 16 > 256 * 256 * n * 1.2) ++bad;
  }
  printf(bad ? "FAIL %d\n" : "OK\n", bad);
  return bad != 0;
}
"""


def test_rods_host(tmp_path):
    src, exe = tmp_path / "r.cpp", tmp_path / "r"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", str(exe), str(src)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr


SHAPES = [(70, 9, 2), (33, 20, 3), (64, 17, 5), (97, 18, 7), (40, 33, 9), (66, 2, 31), (95, 3, 18), (130, 5, 20), (2, 40, 2)]


@pytest.mark.gpu
@pytest.mark.parametrize("mdt,hi,bins", [(np.uint8, 255, 32), (np.uint16, 4095, 128), (np.uint16, 65535, 200)])
def test_thin_and_ragged(mdt, hi, bins):
    import torch
    from paper_1909_10690_amd import binding as B
    ctx = B.Context(0)
    rng = np.random.default_rng(hi + bins)
    pairs, want = [], []
    for shape in SHAPES:
        f = inputs.random_volume(rng, shape, np.uint8, 0, 255)
        m = inputs.random_volume(rng, shape, mdt, 0, hi)
        mats = np.concatenate([inputs.random_affines(rng, 4, shape, rot=4, trans=0.7),
                               inputs.random_affines(rng, 3, shape, rot=90, trans=2)])
        F, M, tr = B.Volume.from_numpy(f, 0, 255), B.Volume.from_numpy(m, 0, hi), torch.from_numpy(mats).cuda()
        oF, oM = oracle.volume(f, 0, 255), oracle.volume(m, 0, hi)
        print(f"rods {shape} {np.dtype(mdt).name} {bins} bins", flush=True)
        for clamp in (0, 1):
            omi, oov, oh = oracle.eval_hard(oF, oM, mats, bins, (1.0,), boundary=clamp, want_hist=True)
            mi, ov, h = ctx.eval(F, M, tr, bins, (1.0,), flags=clamp | B.COMPACT_SLABS, want_hist=True)
            torch.cuda.synchronize()
            assert np.array_equal(h.cpu().numpy().astype(np.uint32), oh), (shape, clamp)
            assert np.array_equal(ov.cpu().numpy(), oov)
            if clamp == 0:
                pairs.append((F, M, tr))
                want.append(omi)
    got = ctx.eval_pairs(pairs, bins, (1.0,)).cpu().numpy()
    w = np.concatenate(want)
    assert np.all(np.abs(got - w) <= 1e-12 * np.maximum(1.0, np.abs(w)))
    ctx.close()
