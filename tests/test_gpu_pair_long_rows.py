"""The potential link search with the grid where rows are long: boxes that meet a
given number of others, around the 32 slots kept for the fill, whole rounds of 64
lanes and the 1,024 that a wave sorts in LDS.  The list is the oracle's, in order,
and the all-pairs search's."""
import numpy as np
import pytest

import oracle
import paper_2106_12655_amd as lk_mod
from paper_2106_12655_amd import inputs as I

pytestmark = pytest.mark.gpu

LENGTHS = [31, 32, 33, 34, 35, 36, 63, 64, 65, 127, 128, 129, 257, 1021, 1022, 1023, 1024, 1025,
           1026, 1400]


def _box(lo, side):
    lo = np.asarray(lo, float)
    return np.stack([lo, lo + side * np.array([1, 0.5, 0]), lo + side, lo + side * np.array([0, 0.5, 1])])


def _scene(dtype, seed):
    """A large box at the front for each length, and that many small ones, apart
    from each other, inside it; other large boxes far apart keep all regular."""
    rng = np.random.default_rng(seed)
    large, small = [], []
    for g, m in enumerate(LENGTHS):
        at = np.array([8.0 * g, 0.0, 0.0])
        large.append(_box(at, 1.0))
        cells = rng.choice(14 ** 3, m, replace=False)
        for c in cells:
            small.append(_box(at + 0.01 + 0.07 * np.array([c % 14, c // 14 % 14, c // 196]), 0.05))
    for k in range(4000):
        small.append(_box([8.0 * (k % 80), 8.0 + 8.0 * (k // 80), 30.0], 1.0))
    loops = [large[k] for k in rng.permutation(len(large))] + \
            [small[k] for k in rng.permutation(len(small))]
    return I._pack(loops, dtype, {}, "rows", 0)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_long_rows_in_order(ctx, dtype):
    import torch
    ls = _scene(dtype, 4)
    xyz, off = torch.from_numpy(ls.xyz).cuda(), torch.from_numpy(ls.offsets).cuda()
    want = oracle.aabb_pairs(ls.xyz, ls.offsets)
    assert sorted(np.bincount(want[:, 0])) == LENGTHS
    try:
        for method in (2, 1, 0):
            ctx.set_option(lk_mod._lib.OPT_PAIR_SEARCH, method)
            got = ctx.build_pairs(xyz, off).cpu().numpy()
            print("method %d: %d pairs" % (method, len(got)), flush=True)
            assert np.array_equal(got, want), method
    finally:
        ctx.set_option(lk_mod._lib.OPT_PAIR_SEARCH, 0)


def test_dense_rows_in_order(ctx):
    """Every box meets some hundred others, in many buckets."""
    import torch
    rng = np.random.default_rng(9)
    loops = [_box(rng.uniform(0, 3, 3), rng.uniform(0.3, 1.0)) for _ in range(3000)]
    ls = I._pack(loops, np.float64, {}, "dense", 0)
    want = oracle.aabb_pairs(ls.xyz, ls.offsets)
    xyz, off = torch.from_numpy(ls.xyz).cuda(), torch.from_numpy(ls.offsets).cuda()
    got = ctx.build_pairs(xyz, off).cpu().numpy()
    print("%d pairs, longest row %d" % (len(want), np.bincount(want[:, 0]).max()), flush=True)
    assert np.array_equal(got, want)
