"""GPU parity of brick sweeps of few transforms, which read rows of octs up to
six transforms and tiles beyond (16-byte records), on one workspace, with the
preparation kept and made anew; histograms bit-exact against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_1909_10690_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mdt,hi", [(np.uint8, 255), (np.uint16, 4095), (np.int16, 30000)])
@pytest.mark.parametrize("shape", [(6, 4, 2), (70, 33, 17), (100, 64, 30)])
def test_few_in_bricks(mdt, hi, shape):
    import torch
    from paper_1909_10690_amd import binding as B
    rng = np.random.default_rng(sum(shape))
    f, m = inputs.random_volume(rng, shape, np.uint8, 0, 255), inputs.random_volume(rng, shape, mdt, 0, hi)
    mats = inputs.random_affines(rng, 8, shape, rot=70, trans=1)
    _, oov, oh = oracle.eval_hard(oracle.volume(f, 0, 255), oracle.volume(m, 0, hi), mats, 40, (1.0,), boundary=0,
                                  want_hist=True)
    ctx = B.Context(0)
    F, M = B.Volume.from_numpy(f, 0, 255), B.Volume.from_numpy(m, 0, hi)
    ws = torch.zeros(ctx.workspace_size(F, M, 8, 40, 1, B.COMPACT_SLABS), dtype=torch.uint8, device="cuda")
    for n in (1, 6, 7, 6, 8, 2):
        for keep in (0, B.VOLUMES_UNCHANGED, 0):
            print(f"few in bricks {shape} {np.dtype(mdt).name} n={n} keep={keep}", flush=True)
            _, ov, h = ctx.eval(F, M, torch.from_numpy(mats[:n]).cuda(), 40, flags=B.COMPACT_SLABS | keep,
                                want_hist=True, workspace=ws)
            torch.cuda.synchronize()
            assert np.array_equal(h.cpu().numpy().astype(np.uint32), oh[:n])
            assert np.array_equal(ov.cpu().numpy(), oov[:n])
    ctx.close()
