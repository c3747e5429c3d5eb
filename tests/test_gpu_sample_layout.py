"""GPU parity of sampled Parzen calls on both moving layouts, at sizes where the
limit between them (tests/test_sample_layout_host.py) lies below the rise of the
turned batch: against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_1909_10690_amd import inputs
from paper_1909_10690_amd import transforms as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mdt,hi,ms", [(np.uint8, 255, (101, 100, 93)), (np.uint16, 65535, (120, 101, 90)),
                                       (np.float32, 1, (130, 101, 101))])
@pytest.mark.parametrize("fraction", [0.4, 1.0])
def test_both_layouts(mdt, hi, ms, fraction):
    import torch
    from paper_1909_10690_amd import binding as B
    rng = np.random.default_rng(ms[0])
    fs = (64, 60, 50)
    f, m = inputs.random_volume(rng, fs, np.uint8, 0, 255), inputs.random_volume(rng, ms, mdt, 0, hi)
    turned = inputs.random_affines(rng, 24, fs, rot=60, trans=2)
    for r in range(3):  # over the whole moving volume
        turned[:, 4 * r:4 * r + 3] *= 2.0
    shifts = np.stack([T.translation((0.25 * k, 1 - 0.5 * k, k % 5)) for k in range(24)]).reshape(-1, 12)
    ctx = B.Context(0)
    F, M = B.Volume.from_numpy(f, 0, 255), B.Volume.from_numpy(m, 0, hi)
    for mats in (shifts, turned):
        print(f"sampled layouts {np.dtype(mdt).name} {ms} fraction={fraction}", flush=True)
        mi, ov, _ = ctx.eval_sampled(F, M, torch.from_numpy(mats).cuda(), 16, (1.0, 1.5), fraction=fraction,
                                     flags=B.HIST_PARZEN)
        omi, on = oracle.eval_parzen(oracle.volume(f, 0, 255), oracle.volume(m, 0, hi), mats, 16, (1.0, 1.5),
                                     boundary=0, sample=(fraction, 0))
        torch.cuda.synchronize()
        assert np.array_equal(ov.cpu().numpy(), on)
        err = np.abs(mi.cpu().numpy() - omi) / np.maximum(1.0, np.abs(omi))
        assert err.max() <= 1e-6, err.max()
    ctx.close()
