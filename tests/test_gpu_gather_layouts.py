"""GPU parity of the moving volume's gather layouts at their edges: volumes
of the smallest size, faces hit exactly (where a gather reads past the row,
slice or volume with weight 0) and unaligned sources, against the CPU oracle.
Hard histograms are bit-exact; Parzen MI within 1e-6 relative."""
import numpy as np
import pytest

import oracle
from paper_1909_10690_amd import inputs
from paper_1909_10690_amd import transforms as T

pytestmark = pytest.mark.gpu

RANGES = {np.uint8: (0, 255), np.uint16: (7, 4000), np.int16: (-1000, 1500), np.float32: (0.1, 0.9)}


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_1909_10690_amd import binding as B
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = B.Context(0)
    yield c
    c.close()


def edge_transforms(shape, rng):
    """Identity, faces hit exactly, a half step past each face, mirrors and
    quarter turns about the centre, one affine."""
    n = np.asarray(shape, dtype=float)
    c = T.fixed_centre(shape)
    mats = [T.translation((0, 0, 0)), T.translation((1, 0, 0)), T.translation((0, -1, 0)), T.translation((0, 0, 1)),
            T.translation((0.5, -0.5, 0.25)), T.translation(tuple(n - 1)), T.translation(tuple(1 - n)),
            T.centred_matrix(np.diag([-1.0, 1.0, 1.0]), (0, 0, 0), c),
            T.centred_matrix(np.array([[0.0, 0, 1], [0, 1, 0], [-1, 0, 0]]), (0, 0, 0), c)]
    return np.concatenate([np.stack(mats).reshape(-1, 12), inputs.random_affines(rng, 1, shape, rot=25, trans=1)])


def device_volume(arr, lo, hi, shift):
    """The volume on the device, its data `shift` elements off an aligned
    address."""
    import torch
    from paper_1909_10690_amd import binding as B
    t = torch.from_numpy(np.ascontiguousarray(arr))
    buf = torch.zeros(t.numel() + shift, dtype=t.dtype, device="cuda")
    v = buf[shift:].view(t.shape)
    v.copy_(t.cuda())
    assert v.is_contiguous()
    return B.Volume(v, lo, hi)


SHAPES = [(2, 2, 2), (5, 3, 2), (17, 4, 3), (33, 19, 6)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("mdt,shift", [(np.uint8, 0), (np.uint8, 3), (np.uint16, 1), (np.int16, 0), (np.float32, 1)])
@pytest.mark.parametrize("clamp", [0, 1])
def test_sampled_parzen_copy(ctx, shape, mdt, shift, clamp):
    """The plain copy of sampled Parzen calls, every voxel kept."""
    import torch
    from paper_1909_10690_amd import binding as B
    rng = np.random.default_rng(sum(shape) + shift)
    f = inputs.random_volume(rng, shape, np.uint8, 0, 255)
    m = inputs.random_volume(rng, shape, mdt, *RANGES[mdt])
    mats, q = edge_transforms(shape, rng), (1.0, 1.5)
    print(f"sampled Parzen copy shape={shape} moving={np.dtype(mdt).name} shift={shift} clamp={clamp}", flush=True)
    lo, hi = RANGES[mdt]
    mi, ov, _ = ctx.eval_sampled(device_volume(f, 0, 255, 0), device_volume(m, lo, hi, shift),
                                 torch.from_numpy(mats).cuda(), 16, q, fraction=1.0, flags=clamp | B.HIST_PARZEN)
    omi, on = oracle.eval_parzen(oracle.volume(f, 0, 255), oracle.volume(m, lo, hi), mats, 16, q, boundary=clamp,
                                 sample=(1.0, 0))
    torch.cuda.synchronize()
    assert np.array_equal(ov.cpu().numpy(), on)
    err = np.abs(mi.cpu().numpy() - omi) / np.maximum(1.0, np.abs(omi))
    assert err.max() <= 1e-6, err.max()


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("mdt,mr,shift", [(np.uint8, (0, 255), 5), (np.uint8, (9, 200), 0), (np.uint16, (0, 65535), 0),
                                          (np.int16, (-1000, 1500), 1)])
@pytest.mark.parametrize("clamp", [0, 1])
def test_few_transforms_use_the_copy(ctx, shape, mdt, mr, shift, clamp):
    """Batches of 1 and 4 (the plain copy) and of 5 and more (octs)."""
    import torch
    rng = np.random.default_rng(sum(shape) + shift)
    f = inputs.random_volume(rng, shape, np.uint8, 0, 255)
    m = inputs.random_volume(rng, shape, mdt, *(mr if mdt != np.uint8 else (0, 255)))
    mats, q = edge_transforms(shape, rng), (1.0, 0.5)
    print(f"copy layout shape={shape} moving={np.dtype(mdt).name} range={mr} clamp={clamp}", flush=True)
    F, M = device_volume(f, 0, 255, 0), device_volume(m, *mr, shift)
    omi, oov, oh = oracle.eval_hard(oracle.volume(f, 0, 255), oracle.volume(m, *mr), mats, 30, q, boundary=clamp,
                                    want_hist=True)
    for sel in ([0], [4], [1, 2, 3, 9], [5, 6, 7, 8], list(range(5)), list(range(10))):
        mi, ov, h = ctx.eval(F, M, torch.from_numpy(mats[sel]).cuda(), 30, q, flags=clamp, want_hist=True)
        torch.cuda.synchronize()
        assert np.array_equal(h.cpu().numpy().astype(np.uint32), oh[sel]), sel
        assert np.array_equal(ov.cpu().numpy(), oov[sel])
        assert np.all(np.abs(mi.cpu().numpy() - omi[sel]) <= 1e-12 * np.maximum(1.0, np.abs(omi[sel])))


def test_preparation_switches_layout(ctx):
    """Calls on one workspace that prepare the copy, prepare octs and reuse
    them (MI_VOLUMES_UNCHANGED), eager and as graphs: every result is that of
    a fresh call.  (The workspace's regions lie elsewhere for 1 and for 8
    transforms, so a preparation serves calls of its own batch size only.)"""
    import torch
    from paper_1909_10690_amd import binding as B
    rng = np.random.default_rng(3)
    shape = (40, 31, 22)
    F = device_volume(inputs.random_volume(rng, shape, np.uint8, 0, 255), 0, 255, 0)
    M = device_volume(inputs.random_volume(rng, shape, np.uint16, 0, 4095), 0, 4095, 0)
    tr = torch.from_numpy(inputs.random_affines(rng, 8, shape)).cuda()
    one, q = tr[2:3].contiguous(), (1.0,)
    want = {1: ctx.eval(F, M, one, 64, q, want_hist=True)[2], 8: ctx.eval(F, M, tr, 64, q, want_hist=True)[2]}
    ws = torch.empty(ctx.workspace_size(F, M, 8, 64, 1), dtype=torch.uint8, device="cuda")
    out = {n: torch.empty((n, 1), dtype=torch.float64, device="cuda") for n in (1, 8)}
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    same = B.VOLUMES_UNCHANGED
    for n, flags in [(1, 0), (1, same), (1, same), (1, 0), (8, same), (1, B.USE_GRAPH), (8, same), (8, B.USE_GRAPH),
                     (1, same), (1, 0), (1, B.USE_GRAPH), (1, same)]:
        x = one if n == 1 else tr
        with torch.cuda.stream(side):
            mi, _, h = ctx.eval(F, M, x, 64, q, flags=flags, want_hist=True, out=out[n], workspace=ws, stream=side)
        side.synchronize()
        assert torch.equal(h, want[n]), (n, flags)


@pytest.mark.parametrize("nx", [15, 63, 64, 65, 79, 128, 150])
@pytest.mark.parametrize("hi,bins", [(255, 128), (16383, 128), (16383, 129), (16384, 64), (65535, 256), (4095, 2),
                                     (4095, 97)])
def test_sweep_runs_and_records(ctx, nx, hi, bins):
    """Rows of and around whole 64-voxel runs; moving ranges on both sides of
    each record form (8-bit corners, differences up to 2^14, 16-bit corners);
    bin counts on both sides of the 16-bit counters, thin slabs and bricks."""
    import torch
    from paper_1909_10690_amd import binding as B
    shape = (nx, 9, 6)
    rng = np.random.default_rng(nx + hi + bins)
    dt = np.uint8 if hi == 255 else np.uint16
    f = inputs.random_volume(rng, shape, np.uint8, 0, 255)
    m = inputs.random_volume(rng, shape, dt, 0, hi)
    mats = edge_transforms(shape, rng)
    print(f"runs nx={nx} hi={hi} bins={bins}", flush=True)
    F, M = device_volume(f, 0, 255, 1), device_volume(m, 0, hi, 0)
    for clamp in (0, 1):
        omi, oov, oh = oracle.eval_hard(oracle.volume(f, 0, 255), oracle.volume(m, 0, hi), mats, bins, (1.0,),
                                        boundary=clamp, want_hist=True)
        for flags in (clamp, clamp | B.COMPACT_SLABS):
            mi, ov, h = ctx.eval(F, M, torch.from_numpy(mats).cuda(), bins, (1.0,), flags=flags, want_hist=True)
            torch.cuda.synchronize()
            assert np.array_equal(h.cpu().numpy().astype(np.uint32), oh), flags
            assert np.array_equal(ov.cpu().numpy(), oov)
            assert np.all(np.abs(mi.cpu().numpy() - omi) <= 1e-12 * np.maximum(1.0, np.abs(omi)))


TILED = [(2, 2, 2), (4, 2, 2), (6, 4, 2), (16, 4, 6), (64, 10, 8), (84, 6, 14)]  # whole tiles, no padding


@pytest.mark.parametrize("shape", TILED)
@pytest.mark.parametrize("mdt,hi,bins", [(np.uint8, 255, 64), (np.uint8, 200, 256), (np.uint16, 4095, 128),
                                         (np.uint16, 65535, 129)])
def test_brick_tiles(ctx, shape, mdt, hi, bins):
    """Bricks over tiles of octs: moving volumes of one tile and more, fixed
    volumes of their extents and ragged ones around a rod and a run."""
    import torch
    from paper_1909_10690_amd import binding as B
    rng = np.random.default_rng(sum(shape) + hi + bins)
    m = inputs.random_volume(rng, shape, mdt, 0, hi)
    for fs in (shape, (67, 5, 3), (17, 9, 2)):
        f = inputs.random_volume(rng, fs, np.uint8, 0, 255)
        mats = edge_transforms(fs, rng)
        print(f"tiles moving={shape} fixed={fs} hi={hi} bins={bins}", flush=True)
        F, M = device_volume(f, 0, 255, 1), device_volume(m, 0, hi, 0)
        for clamp in (0, 1):
            omi, oov, oh = oracle.eval_hard(oracle.volume(f, 0, 255), oracle.volume(m, 0, hi), mats, bins, (1.0,),
                                            boundary=clamp, want_hist=True)
            mi, ov, h = ctx.eval(F, M, torch.from_numpy(mats).cuda(), bins, (1.0,), flags=clamp | B.COMPACT_SLABS,
                                 want_hist=True)
            torch.cuda.synchronize()
            assert np.array_equal(h.cpu().numpy().astype(np.uint32), oh), (fs, clamp)
            assert np.array_equal(ov.cpu().numpy(), oov)
            assert np.all(np.abs(mi.cpu().numpy() - omi) <= 1e-12 * np.maximum(1.0, np.abs(omi)))


@pytest.mark.parametrize("mdt,lo,hi,shift", [(np.uint8, 0, 255, 0), (np.uint8, 0, 255, 3), (np.uint8, 9, 200, 1),
                                             (np.int16, -100, 100, 0), (np.uint16, 0, 65535, 1)])
@pytest.mark.parametrize("bins", [32, 128, 200])
def test_pair_tiles(ctx, mdt, lo, hi, shift, bins):
    """Padded tiles of pairs: moving extents on both sides of whole tiles,
    rows shorter than one, unaligned sources."""
    import torch
    rng = np.random.default_rng(hi + shift + bins)
    shapes = [(2, 2, 2), (3, 5, 2), (4, 3, 3), (5, 2, 7), (6, 6, 5), (7, 4, 4), (33, 19, 6), (64, 8, 8), (130, 9, 5)]
    pairs, want = [], []
    for i, ms in enumerate(shapes):
        fs = shapes[(i + 3) % len(shapes)]
        f = inputs.random_volume(rng, fs, np.uint8, 0, 255)
        m = inputs.random_volume(rng, ms, mdt, *((0, 255) if mdt == np.uint8 else (lo, hi)))
        mats = edge_transforms(fs, rng)
        pairs.append((device_volume(f, 0, 255, shift), device_volume(m, lo, hi, shift), torch.from_numpy(mats).cuda()))
        want.append([oracle.eval_hard(oracle.volume(f, 0, 255), oracle.volume(m, lo, hi), mats, bins, (1.0,),
                                      boundary=c)[0] for c in (0, 1)])
    for clamp in (0, 1):
        print(f"pair tiles {np.dtype(mdt).name} {lo}..{hi} bins={bins} clamp={clamp}", flush=True)
        got = ctx.eval_pairs(pairs, bins, (1.0,), flags=clamp)
        torch.cuda.synchronize()
        w = np.concatenate([x[clamp] for x in want])
        assert np.all(np.abs(got.cpu().numpy() - w) <= 1e-12 * np.maximum(1.0, np.abs(w)))


@pytest.mark.parametrize("shape", [(64, 64, 64), (68, 64, 61), (80, 64, 64)])
@pytest.mark.parametrize("n", [64, 4150])
def test_order_around_the_l2(ctx, shape, n):
    """Moving layouts of 4 MiB (batch order) and of a little more (processing
    order, one sorted block and two): every histogram, overlap and MI equals
    that of the same transform in a batch of 50, which keeps the batch
    order; the slices of the reduction differ, so MI within 1e-12."""
    import torch
    rng = np.random.default_rng(n + shape[0])
    V = device_volume(inputs.random_volume(rng, shape, np.uint16, 0, 4095), 0, 4095, 0)
    mats = torch.from_numpy(inputs.random_affines(rng, n, shape, rot=25.0, trans=4.0)).cuda()
    print(f"order shape={shape} n={n}", flush=True)
    mi, ov, h = ctx.eval(V, V, mats, 32, (1.0, 1.5), want_hist=True)
    for t0 in sorted({0, 50, n // 2, n - 50}):
        mi_s, ov_s, h_s = ctx.eval(V, V, mats[t0:t0 + 50], 32, (1.0, 1.5), want_hist=True)
        torch.cuda.synchronize()
        assert torch.equal(h[t0:t0 + 50], h_s) and torch.equal(ov[t0:t0 + 50], ov_s), t0
        assert torch.all((mi[t0:t0 + 50] - mi_s).abs() <= 1e-12 * torch.clamp(mi_s.abs(), min=1.0))


@pytest.mark.parametrize("mdt,shape", [(np.uint16, (101, 100, 93)), (np.uint8, (160, 101, 90)),
                                       (np.float32, (130, 129, 125))])
@pytest.mark.parametrize("clamp", [0, 1])
def test_sampled_parzen_records(ctx, mdt, shape, clamp):
    """Sampled Parzen batches on volumes large enough for the choice of the
    moving layout: shifts (the copy), wide turns (records) and both."""
    import torch
    from paper_1909_10690_amd import binding as B
    rng = np.random.default_rng(shape[0])
    lo, hi = RANGES[mdt]
    fs = (40, 33, 21)
    f = inputs.random_volume(rng, fs, np.uint8, 0, 255)
    m = inputs.random_volume(rng, shape, mdt, lo, hi)
    turned = inputs.random_affines(rng, 4, fs, rot=60, trans=2)
    turned[:, :3] *= 3.0  # over the whole moving volume
    turned[:, 4:7] *= 3.0
    turned[:, 8:11] *= 3.0
    shifts = np.stack([T.translation(v) for v in ((0, 0, 0), (3, -2.5, 1), (0.5, 4, 9))]).reshape(-1, 12)
    F, M = device_volume(f, 0, 255, 0), device_volume(m, lo, hi, 1)
    for mats in (shifts, turned, np.concatenate([shifts, turned])):
        print(f"sampled Parzen records {np.dtype(mdt).name} {shape} clamp={clamp} n={len(mats)}", flush=True)
        mi, ov, _ = ctx.eval_sampled(F, M, torch.from_numpy(mats).cuda(), 16, (1.0, 1.5), fraction=0.6,
                                     flags=clamp | B.HIST_PARZEN)
        omi, on = oracle.eval_parzen(oracle.volume(f, 0, 255), oracle.volume(m, lo, hi), mats, 16, (1.0, 1.5),
                                     boundary=clamp, sample=(0.6, 0))
        torch.cuda.synchronize()
        assert np.array_equal(ov.cpu().numpy(), on)
        err = np.abs(mi.cpu().numpy() - omi) / np.maximum(1.0, np.abs(omi))
        assert err.max() <= 1e-6, err.max()
