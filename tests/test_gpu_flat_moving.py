"""GPU parity on moving volumes of very many short rows (2 x 4096 x 4096): a
workgroup for each row would wrap the preparation's launch, so the octs are
packed in turns.  Histograms bit-exact against the CPU oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,hi", [(np.uint16, 4095), (np.uint16, 65535), (np.uint8, 255)])
def test_rows_taken_in_turns(dtype, hi):
    import torch
    from paper_1909_10690_amd import binding as B
    rng = np.random.default_rng(hi)
    f = rng.integers(0, 256, (20, 30, 40), dtype=np.uint8)
    m = rng.integers(0, hi + 1, (4096, 4096, 2), dtype=dtype)
    n = 6
    M = np.zeros((n, 3, 4))
    M[:, 0, 0], M[:, 1, 1], M[:, 2, 2] = 1 / 39, 4095 / 29, 4095 / 19  # the fixed grid spans the moving one
    M[:, :, :3] *= rng.uniform(0.97, 1.0, (n, 3, 3))
    M[:, :, 3] = rng.uniform(0, 1, (n, 3)) * (0.02, 60, 60)
    M = M.reshape(n, 12)
    print(f"flat moving {m.shape} {np.dtype(dtype).name} hi={hi}", flush=True)
    ctx = B.Context(0)
    F, V = B.Volume.from_numpy(f, 0, 255), B.Volume.from_numpy(m, 0, hi)
    tr = torch.from_numpy(M).cuda()
    oF, oM = oracle.volume(f, 0, 255), oracle.volume(m, 0, hi)
    _, oov, oh = oracle.eval_hard(oF, oM, M, 40, (1.0,), want_hist=True)
    assert oov.min() > f.size // 2
    _, ov, h = ctx.eval(F, V, tr, 40, (1.0,), want_hist=True)
    torch.cuda.synchronize()
    assert np.array_equal(ov.cpu().numpy(), oov)
    assert np.array_equal(h.cpu().numpy().astype(np.uint32), oh)
    _, ov, h = ctx.eval_sampled(F, V, tr, 40, (1.0,), fraction=1.0, want_hist=True)
    torch.cuda.synchronize()
    assert np.array_equal(ov.cpu().numpy(), oov)
    assert np.array_equal(h.cpu().numpy().astype(np.uint32), oh)
    ctx.close()
