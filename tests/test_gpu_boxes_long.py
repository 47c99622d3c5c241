"""Boxes of scenes with so many loops that 16 lanes take one: loops around the
length from which a whole wave takes it, at every place in a wave, among short
and empty ones."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("case", ["few long", "all long in a part", "one longest", "edges"])
def test_boxes_of_long_loops(ctx, case, dtype):
    import torch
    rng = np.random.default_rng(len(case))
    n = 8195
    sizes = rng.integers(3, 9, n)
    if case == "few long":
        sizes[rng.choice(n, 300, replace=False)] = rng.integers(1500, 3000, 300)
    elif case == "all long in a part":
        sizes[:] = rng.integers(40, 60, n)
        sizes[3000:3200] = rng.integers(2049, 2100, 200)
    elif case == "one longest":
        sizes[8194] = 300001
        sizes[0:8] = (3000, 3, 0, 5, 3, 2500, 2060, 4000)
    else:
        sizes[1000:1064] = np.tile([2047, 2048, 2049, 0, 15, 16, 17, 2050], 8)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    xyz = (rng.uniform(0, 40, (n, 3))[np.repeat(np.arange(n), sizes)]
           + rng.uniform(-0.5, 0.5, (off[-1], 3))).astype(dtype)
    # the extreme vertex of each loop at either end or in the middle
    some = np.nonzero(sizes > 3)[0]
    xyz[off[some] + (sizes[some] - 1) * rng.integers(0, 3, len(some)) // 2] += dtype(0.7)
    want = oracle.aabb_pairs(xyz, off)
    got = ctx.build_pairs(torch.from_numpy(xyz).cuda(), torch.from_numpy(off).cuda()).cpu().numpy()
    print(case, dtype.__name__, len(want), "pairs, longest loop", sizes.max(), flush=True)
    assert np.array_equal(got, want)
