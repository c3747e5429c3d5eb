"""GPU tests of the MI reduction at the edges of its slicing: bin counts
around 16 (one slice) and 8 s (slices of 8 and 9 rows), batches of one slice
and of many, one entropy and sixteen, transforms without overlap, against the
CPU oracle (hard MI within 1e-12, Parzen MI within 1e-6 for q >= 1, where an
fp32 weight's error is not magnified by the smallest masses; overlaps
exact)."""
import numpy as np
import pytest

import oracle
from paper_1909_10690_amd import inputs

pytestmark = pytest.mark.gpu

Q16 = (1.0, 0.5, 0.8, 0.999, 1.001, 1.2, 1.5, 2.0, 2.5, 3.0, 0.25, 0.1, 1.1, 1.3, 1.7, 4.0)


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_1909_10690_amd import binding as B
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = B.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("bins,n,q", [(2, 1, Q16), (5, 3, (1.0,)), (15, 7, Q16), (16, 1, Q16), (17, 600, (1.0,)),
                                      (17, 3, Q16), (23, 513, (1.5,)), (33, 512, (1.0, 2.0)), (63, 1, Q16),
                                      (100, 11, Q16), (129, 2, Q16), (255, 1, Q16), (256, 5, Q16),
                                      (256, 520, (1.0,))])
@pytest.mark.parametrize("parzen", [False, True])
def test_reduction_slices(ctx, bins, n, q, parzen):
    import torch
    from paper_1909_10690_amd import binding as B
    if parzen and bins < 8:
        pytest.skip("Parzen windows need more bins")
    if parzen and len(q) == 16:
        q = tuple(1 + 0.2 * i for i in range(16))
    rng = np.random.default_rng(bins * 1000 + n)
    shape = (13, 9, 6)
    f = inputs.random_volume(rng, shape, np.uint8, 0, 255)
    m = inputs.random_volume(rng, shape, np.uint16, 0, 4095)
    mats = inputs.random_affines(rng, n, shape, trans=2)
    mats[n // 2] = [1, 0, 0, 1000, 0, 1, 0, 0, 0, 0, 1, 0]  # no overlap
    if n > 2:
        mats[1] = [1, 0, 0, 12, 0, 1, 0, 8, 0, 0, 1, 5]  # one voxel
    print(f"reduction bins={bins} n={n} entropies={len(q)} parzen={parzen}", flush=True)
    V = [B.Volume(torch.from_numpy(a).cuda(), 0, hi) for a, hi in ((f, 255), (m, 4095))]
    run = oracle.eval_parzen if parzen else oracle.eval_hard
    for form, pseudo in ((0, B.TSALLIS_ADDITIVE), (1, B.TSALLIS_PSEUDOADDITIVE)) if n < 20 else ((0, 0),):
        want = run(oracle.volume(f, 0, 255), oracle.volume(m, 0, 4095), mats, bins, q, boundary=0, form=form)
        mi, ov, _ = ctx.eval(*V, torch.from_numpy(mats).cuda(), bins, q,
                             flags=pseudo | (B.HIST_PARZEN if parzen else 0))
        torch.cuda.synchronize()
        assert np.array_equal(ov.cpu().numpy(), want[1])
        err = np.abs(mi.cpu().numpy() - want[0]) / np.maximum(1.0, np.abs(want[0]))
        assert err.max() <= (1e-6 if parzen else 1e-12), err.max()
