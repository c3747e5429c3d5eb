"""Brick sweeps of volumes long in x, whose slabs are dealt to the XCDs in turn: a
CPU test that every slab is dealt once and that the XCDs share the rods of every x
segment, and GPU parity at the rule's edges, bit-exact against the CPU oracle."""
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_1909_10690_amd import inputs

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1909_10690_amd", "csrc")

PROGRAM = r"""
#include "plan.h"
#include <stdio.h>
#include <vector>
using namespace gemi;
int main() {
  int bad = 0;
  for (uint32_t chunks = 8; chunks <= 2048; chunks += 8) {
    std::vector<int> seen(chunks, 0);
    for (uint32_t c = 0; c < chunks; ++c) {
      const uint32_t d = dealt_slab(c, chunks);
      if (d >= chunks) { ++bad; continue; }
      ++seen[d];
      bad += d % 8 != c / (chunks / 8);  // XCD x takes slabs x, x + 8, ...
    }
    for (int v : seen) bad += v != 1;
  }
  // 512x512x48 in 64 slabs: each XCD has rods of every x segment; by eighths, of one
  const Rods r = rods_for(512, 512, 48);
  for (int dealt = 0; dealt < 2; ++dealt)
    for (uint32_t xcd = 0; xcd < 8; ++xcd) {
      uint32_t segments = 0;
      for (uint32_t c = 8 * xcd; c < 8 * xcd + 8; ++c) {
        RodWalk w;
        w.init(r, 512, 48, 64, dealt ? dealt_slab(c, 64) : c, 0);
        for (; w.u < w.u1; w.next(16)) segments |= 1u << w.xs;
      }
      bad += dealt ? segments != (1u << r.segments) - 1 : (segments & (segments - 1)) != 0;
    }
  bad += !deal_slabs(512, 512, 48) || !deal_slabs(40, 20, 90) || deal_slabs(256, 256, 180) || deal_slabs(39, 20, 90) || deal_slabs(64, 256, 256);
  printf(bad ? "FAIL %d\n" : "OK\n", bad);
  return bad != 0;
}
"""


def test_dealt_slabs_host(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", str(exe), str(src)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(2, 2, 2), (40, 20, 33), (39, 20, 33), (300, 70, 9), (130, 5, 64)])
@pytest.mark.parametrize("bins,clamp", [(32, 0), (200, 1)])
def test_dealt_slabs(shape, bins, clamp):
    import torch
    from paper_1909_10690_amd import binding as B
    rng = np.random.default_rng(sum(shape))
    f, m = inputs.random_volume(rng, shape, np.uint8, 0, 255), inputs.random_volume(rng, shape, np.uint16, 0, 4095)
    mats = inputs.random_affines(rng, 40, shape, rot=90, trans=1)
    _, oov, oh = oracle.eval_hard(oracle.volume(f, 0, 255), oracle.volume(m, 0, 4095), mats, bins, (1.0,), boundary=clamp,
                                  want_hist=True)
    ctx = B.Context(0)
    F, M = B.Volume.from_numpy(f, 0, 255), B.Volume.from_numpy(m, 0, 4095)
    for n in (40, 3):
        print(f"dealt slabs {shape} bins={bins} clamp={clamp} n={n}", flush=True)
        _, ov, h = ctx.eval(F, M, torch.from_numpy(mats[:n]).cuda(), bins, flags=B.COMPACT_SLABS | clamp, want_hist=True)
        torch.cuda.synchronize()
        assert np.array_equal(h.cpu().numpy().astype(np.uint32), oh[:n])
        assert np.array_equal(ov.cpu().numpy(), oov[:n])
    ctx.close()
