"""GPU tests of the record of what a workspace holds (MI_VOLUMES_UNCHANGED):
a call that may reuse a preparation finds it where the last one put it, or
prepares again.  Histograms are exact and the MI of one batch is summed in a
fixed order, so every result equals that of a fresh workspace bit for bit."""
import numpy as np
import pytest

from paper_1909_10690_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_1909_10690_amd import binding as B
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = B.Context(0)
    yield c
    c.close()


def pair_set(seed, n=4, transforms=6):
    import torch
    from paper_1909_10690_amd import binding as B
    rng = np.random.default_rng(seed)
    pairs = []
    for k in range(n):
        shape = tuple(int(e) for e in rng.choice([24, 33, 40], 3))
        pairs.append((B.Volume.from_numpy(inputs.random_volume(rng, shape, np.uint8, 0, 255), 0, 255),
                      B.Volume.from_numpy(inputs.random_volume(rng, shape, np.uint8, 0, 255), 0, 255),
                      torch.from_numpy(inputs.random_affines(rng, transforms, shape, rot=10, trans=3)).cuda()))
    return pairs


def test_pairs_of_other_batch_sizes(ctx):
    """The same pairs on one workspace with fewer and more transforms and
    another number of entropies: the pairs' bins and octs lie elsewhere then."""
    import torch
    from paper_1909_10690_amd import binding as B
    pairs = pair_set(71)
    few = [(f, m, t[:k + 1].contiguous()) for k, (f, m, t) in enumerate(pairs)]
    one, three = (1.0,), (1.0, 0.5, 2.0)
    ws = torch.empty(ctx.pairs_workspace_size(pairs, 40, 3), dtype=torch.uint8, device="cuda")
    calls = [(pairs, one), (few, one), (few, three), (pairs, three), (pairs, one), (few, three)]
    want = [ctx.eval_pairs(p, 40, q).cpu() for p, q in calls]
    for k, (p, q) in enumerate(calls):
        print(f"pairs batch {k}", flush=True)
        got = ctx.eval_pairs(p, 40, q, flags=B.VOLUMES_UNCHANGED, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(got.cpu(), want[k]), k


@pytest.mark.parametrize("shape_line", ["256 1 64 0", "512 0 32 1", "1024 1 64 0"])
def test_graph_then_another_launch_shape(tmp_path, monkeypatch, shape_line):
    """A graph captured under one launch shape (read from a cache file), a
    tuning that may pick another, the graph's call again, then a call that
    reuses what it prepared: the bins' order and the octs' layout follow the
    shape (1024 threads sweep bricks here, 256 and 512 thin slabs, and whichever
    kind the tuning picks, a start from the other changes)."""
    import torch
    from paper_1909_10690_amd import binding as B
    rng = np.random.default_rng(5)
    shape = (64, 32, 24)
    F = B.Volume.from_numpy(inputs.random_volume(rng, shape, np.uint8, 0, 255), 0, 255)
    M = B.Volume.from_numpy(inputs.random_volume(rng, shape, np.uint16, 0, 4000), 0, 4000)
    tr = torch.from_numpy(inputs.random_affines(rng, 8, shape)).cuda()
    path = tmp_path / "tune.txt"
    # class of these volumes: extents, dtype, bins, boundary, 2^3 transforms, 16-bit corners
    path.write_text(f"gemi-tune 64 32 24 64 32 24 1 64 0 3 0 {shape_line}\n")
    assert B.read_tune_cache(str(path))[0]["block"] == int(shape_line.split()[0])
    monkeypatch.setenv("MI_TUNE_CACHE", str(path))
    ctx = B.Context(0)
    want = ctx.eval(F, M, tr, 64)[0].cpu()
    ws = torch.empty(ctx.workspace_size(F, M, 8, 64, 1, B.COMPACT_SLABS), dtype=torch.uint8, device="cuda")
    out, side = torch.empty((8, 1), dtype=torch.float64, device="cuda"), torch.cuda.Stream()

    def graph():
        with torch.cuda.stream(side):
            ctx.eval(F, M, tr, 64, flags=B.COMPACT_SLABS | B.USE_GRAPH, want_overlap=False, out=out, workspace=ws,
                     stream=side)
        side.synchronize()
        assert torch.equal(out.cpu(), want)

    def reuse():
        got = ctx.eval(F, M, tr, 64, flags=B.COMPACT_SLABS | B.VOLUMES_UNCHANGED, workspace=ws)[0]
        torch.cuda.synchronize()
        assert torch.equal(got.cpu(), want)

    torch.cuda.synchronize()
    for _ in range(2):
        graph()
        reuse()
    ctx.tune(F, M, tr, 64, flags=B.COMPACT_SLABS)
    print(f"from {shape_line} tuned to {B.read_tune_cache(str(path))[0]['block']} threads", flush=True)
    for _ in range(2):
        graph()
        reuse()
    ctx.close()


def test_pairs_and_single_calls_share_a_workspace(ctx):
    """Single-pair calls of every kind, and the LDS probe, between pairs calls
    that may reuse their preparation on the same workspace, and the reverse."""
    import torch
    from paper_1909_10690_amd import binding as B
    pairs = pair_set(73)
    F, M, tr = pairs[0]
    same = B.VOLUMES_UNCHANGED
    ws = torch.empty(1 << 26, dtype=torch.uint8, device="cuda")
    want = ctx.eval_pairs(pairs, 40).cpu()
    single = ctx.eval(F, M, tr, 40)[0].cpu()

    def probe():
        ctx._ws, kept = ws, ctx._ws
        ctx.probe_lds_atomics()
        ctx._ws = kept

    others = {"eval": lambda: ctx.eval(F, M, tr, 40, workspace=ws),
              "sampled": lambda: ctx.eval_sampled(F, M, tr, 40, fraction=0.5, workspace=ws),
              "grad": lambda: ctx.grad(F, M, tr, 40, workspace=ws),
              "tune": lambda: ctx.tune(F, M, tr, 40, workspace=ws),
              "probe": probe,
              "eval further in": lambda: ctx.eval(F, M, tr, 40, workspace=ws[4096:])}
    for name, call in others.items():
        print(f"pairs around {name}", flush=True)
        for _ in range(2):
            assert torch.equal(ctx.eval_pairs(pairs, 40, flags=same, workspace=ws).cpu(), want), name
        call()
        assert torch.equal(ctx.eval_pairs(pairs, 40, flags=same, workspace=ws).cpu(), want), name
        assert torch.equal(ctx.eval(F, M, tr, 40, flags=same, workspace=ws)[0].cpu(), single), name
    probe()
    assert torch.equal(ctx.eval(F, M, tr, 40, flags=same, workspace=ws)[0].cpu(), single)
