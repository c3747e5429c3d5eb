"""GPU parity of the pairs' preparation against the CPU oracle: fixed volumes
of every type in whole runs and ragged rows, aligned and not, moving volumes
whose rows end at every place of a tile and of an 8-byte load, in 8-bit and in
16-bit corners.  Counts are exact, so MI within 1e-12 * max(1, |MI|)."""
import numpy as np
import pytest

import oracle
from paper_1909_10690_amd import inputs
from paper_1909_10690_amd import transforms as T

pytestmark = pytest.mark.gpu

RANGES = {np.uint8: (0, 255), np.uint16: (7, 4000), np.int16: (-1000, 1500), np.float32: (0.1, 0.9)}


def device_volume(arr, lo, hi, shift):
    """The volume on the device, its data `shift` elements off an aligned address."""
    import torch
    from paper_1909_10690_amd import binding as B
    t = torch.from_numpy(np.ascontiguousarray(arr))
    buf = torch.zeros(t.numel() + shift, dtype=t.dtype, device="cuda")
    v = buf[shift:].view(t.shape)
    v.copy_(t.cuda())
    return B.Volume(v, lo, hi)


def check(pairs, want, tag):
    import torch
    from paper_1909_10690_amd import binding as B
    print(tag, flush=True)
    ctx = B.Context(0)
    got = ctx.eval_pairs(pairs, 40, (1.0,)).cpu().numpy()
    torch.cuda.synchronize()
    w = np.concatenate(want)
    assert np.all(np.abs(got - w) <= 1e-12 * np.maximum(1.0, np.abs(w)))
    ctx.close()


def mats(shape, rng):
    """Identity, the faces hit exactly, two affines."""
    n = np.asarray(shape, dtype=float)
    m = [T.translation((0, 0, 0)), T.translation((1, -1, 0)), T.translation((0.5, 0.25, -0.5)), T.translation(tuple(n - 2))]
    return np.concatenate([np.stack(m).reshape(-1, 12), inputs.random_affines(rng, 2, shape, rot=8, trans=1)])


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16, np.int16, np.float32])
@pytest.mark.parametrize("shift", [0, 1])
def test_fixed_types_and_rows(dtype, shift):
    import torch
    rng = np.random.default_rng(shift + 11)
    pairs, want = [], []
    for shape in [(16, 16, 9), (64, 8, 6), (96, 5, 5), (2, 9, 70), (15, 20, 9), (63, 9, 5), (65, 17, 3), (130, 6, 4)]:
        f, m = inputs.random_volume(rng, shape, dtype, *RANGES[dtype]), inputs.random_volume(rng, shape, np.uint8, 0, 255)
        tr = mats(shape, rng)
        pairs.append((device_volume(f, *RANGES[dtype], shift), device_volume(m, 0, 255, 0), torch.from_numpy(tr).cuda()))
        want.append(oracle.eval_hard(oracle.volume(f, *RANGES[dtype]), oracle.volume(m, 0, 255), tr, 40, (1.0,))[0])
    check(pairs, want, f"pairs fixed {np.dtype(dtype).name} shift={shift}")


@pytest.mark.parametrize("kind", ["u8", "u8 clamped", "u8 wide", "u16", "i16", "u16 narrow", "mixed"])
@pytest.mark.parametrize("shift", [0, 3])
def test_moving_types_and_row_ends(kind, shift):
    """`wide`: u8 beside a u16 pair, so all octs have 16-bit corners; `narrow`: u16 of a range of 8 bits."""
    import torch
    rng = np.random.default_rng(shift + 23)
    pairs, want = [], []
    for i, shape in enumerate([(2, 2, 2), (3, 2, 3), (4, 5, 2), (5, 3, 4), (6, 6, 3), (7, 2, 5), (8, 4, 4), (9, 7, 2), (33, 5, 6)]):
        dtype, lo, hi = {"u8": (np.uint8, 0, 255), "u8 clamped": (np.uint8, 9, 200), "u8 wide": (np.uint8, 3, 250),
                         "u16": (np.uint16, 7, 60000), "i16": (np.int16, -900, 1500), "u16 narrow": (np.uint16, 100, 355),
                         "mixed": [(np.uint8, 0, 255), (np.uint16, 5, 4000), (np.int16, -50, 700)][i % 3]}[kind]
        if kind == "u8 wide" and i == 0:
            dtype, lo, hi = np.uint16, 0, 4095
        span = (0, 255) if dtype == np.uint8 else (lo, hi)
        f, m = inputs.random_volume(rng, shape, np.uint8, 0, 255), inputs.random_volume(rng, shape, dtype, *span)
        tr = mats(shape, rng)
        pairs.append((device_volume(f, 0, 255, 0), device_volume(m, lo, hi, shift), torch.from_numpy(tr).cuda()))
        want.append(oracle.eval_hard(oracle.volume(f, 0, 255), oracle.volume(m, lo, hi), tr, 40, (1.0,))[0])
    check(pairs, want, f"pairs moving {kind} shift={shift}")
