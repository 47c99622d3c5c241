"""Calls with few pairs: an item per team of waves, and the preparation in pieces.

Beyond two pairs per compute unit a call runs an item per wave instead.  A big
pair (loop A of 128 segments or more, or several items) is summed in the same
order in both, so its value is the same to the last bit; small pairs get other
lanes, and are held to the oracle: FP64 sums of at most 3e6 terms of error below
4e-16 each differ by less than 2e-9, mixed ones give the oracle's integers."""
import numpy as np
import pytest

import oracle
import paper_2106_12655_amd as lk_mod
from paper_2106_12655_amd import _lib

pytestmark = pytest.mark.gpu


def _loop(n, rng):
    t = 2 * np.pi * (np.arange(n) + rng.uniform(0.1, 0.9, n) * (n > 8)) / max(n, 1)
    r = 1.0 + 0.2 * np.sin(3 * t + rng.uniform(0, 6))
    q = np.linalg.qr(rng.normal(size=(3, 3)))[0]
    return np.stack([r * np.cos(t), r * np.sin(t), 0.3 * np.sin(2 * t)], 1) @ q \
        + rng.uniform(-0.8, 0.8, 3)


def _pack(sizes, dtype, seed):
    rng = np.random.default_rng(seed)
    xyz = np.concatenate([_loop(n, rng) for n in sizes]).astype(dtype)
    return xyz, np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)


def _run(ctx, xyz, off, pairs, mode):
    import torch
    out = ctx.direct_sum(xyz, off, torch.from_numpy(np.asarray(pairs, np.int32)).cuda(), mode=mode)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in out]


A_SIZES = [5, 126, 127, 128, 129, 255, 256, 257, 259, 511, 512, 513, 515, 1023, 2048, 2051, 4097]
B_SIZES = [3, 63, 64, 65, 127, 128, 129, 255, 257, 600]


@pytest.mark.parametrize("mode,dtype,options", [
    ("mixed", np.float32, {}), ("mixed", np.float64, {"SEGS_PER_LANE": 2}), ("plain", np.float64, {}),
    ("plain", np.float32, {"TILE_A": 112}), ("mixed", np.float32, {"TILE_A": 16}),
    ("mixed", np.float32, {"TILE_A": 1024, "CHUNK_A": 2048}), ("plain", np.float64, {"TILE_A": 512}),
    ("mixed", np.float64, {"TILE_A": 272, "CHUNK_A": 544, "WAVES_PER_CU": 4})])
def test_teams_sum_in_the_same_order(ctx, mode, dtype, options):
    import torch
    xyz, off = _pack(A_SIZES + B_SIZES, dtype, 3)
    pairs = [(i, len(A_SIZES) + j) for i in range(len(A_SIZES)) for j in range(len(B_SIZES))]
    big = np.array([A_SIZES[i] >= 128 for i, _ in pairs])
    x, o = torch.from_numpy(xyz).cuda(), torch.from_numpy(off).cuda()
    print(mode, dtype.__name__, options, flush=True)
    keys = {k: getattr(_lib, "OPT_" + k) for k in options}
    try:
        for k, v in options.items():
            ctx.set_option(keys[k], v)
        few = _run(ctx, x, o, pairs, mode)
        again = _run(ctx, x, o, pairs, mode)
        many = [t[:len(pairs)] for t in _run(ctx, x, o, pairs * 5, mode)]
    finally:
        for k in options:
            ctx.set_option(keys[k], 0)
    want = oracle.direct_sum(xyz.astype(np.float64), off, np.asarray(pairs, np.int32))[0]
    assert np.array_equal(few[0], again[0])
    assert np.array_equal(few[0][big], many[0][big])
    assert np.array_equal(few[1], many[1]) and np.array_equal(few[2] & ~1, many[2] & ~1)
    assert np.array_equal(few[1], np.rint(want))
    if mode == "plain":
        assert np.abs(few[0] - want).max() < 2e-9


@pytest.mark.parametrize("sizes", [
    [1024, 1024], [1025, 1024], [32] * 1024, [32] * 1023 + [33], [7] * 1025,
    [0, 1, 2, 3, 9000, 0, 0, 5, 40000, 3, 0], [100003, 5], [7] * 3000,
    [3, 0, 2500, 4, 1] * 40], ids=lambda s: "%d-%d" % (len(s), sum(s)))
def test_preparation_in_pieces(ctx, sizes):
    """Flags of loops with a bad vertex or a zero-length segment at the pieces'
    ends equal those of a call with many pairs, which scans a loop per wave."""
    import torch
    xyz, off = _pack(sizes, np.float64, 5)
    n = len(xyz)
    piece = -(-n // 2048)
    rng = np.random.default_rng(len(sizes))
    x = torch.from_numpy(xyz).cuda()
    o = torch.from_numpy(off).cuda()
    loops = np.arange(len(sizes))
    # each of the chosen loops in a pair with the first (both orders of the index)
    chosen = rng.choice(loops, min(len(loops), 250), replace=False)
    pairs = [(int(a), int((a + 1) % max(2, len(loops)))) for a in chosen]
    print(len(sizes), "loops", n, "vertices", flush=True)
    for plant in range(6):
        y = x.clone()
        at = {0: [], 1: [piece * (n // piece // 2)], 2: [piece * 3 - 1, n - 1],
              3: [0], 4: [piece * k for k in range(1, n // piece, 97)], 5: [n // 2, n // 3]}[plant]
        for v in at:
            if plant % 2:
                y[v] = float("nan") if plant == 1 else float("inf")
            else:  # repeats the vertex before it in its loop: no length
                l = int(np.searchsorted(off, v, "right")) - 1
                y[v] = y[v - 1 if v > off[l] else off[l + 1] - 1]
        few = _run(ctx, y, o, pairs, "mixed")
        many = [t[:len(pairs)] for t in _run(ctx, y, o, pairs * (1 + 600 // len(pairs)), "mixed")]
        assert np.array_equal(few[2] & ~1, many[2] & ~1), plant
        assert np.array_equal(few[1], many[1]), plant
