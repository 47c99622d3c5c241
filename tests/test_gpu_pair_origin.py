"""The grid search's origin: scenes on every side of the coordinate origin, with
loops or single vertices thrown far off in either direction.  Whatever is binned
or tested against all, the list is the oracle's."""
import numpy as np
import pytest

import oracle
import paper_2106_12655_amd as lk_mod
from paper_2106_12655_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("centre", [(0, 0, 0), (-1e3, 2e3, -3e3), (1e5, -1e5, 0)])
@pytest.mark.parametrize("thrown", [(), (-1e13,), (1e13,), (-1e13, 1e13, -1e15), ("vertex", -1e20),
                                    ("vertex", 1e20)])
def test_thrown_loops(ctx, thrown, centre, dtype):
    import torch
    rng = np.random.default_rng(len(thrown) + 3)
    ring = I.circle(6)
    loops = [ring @ I.random_rotation(rng).T * rng.uniform(0.3, 0.6) + rng.uniform(-8, 8, 3) + centre
             for _ in range(2500)]
    if thrown[:1] == ("vertex",):
        loops[0][2, 1] = thrown[1]
        loops[1700][4] = thrown[1]
    else:
        for k, x in enumerate(thrown):
            loops[700 * k] = loops[700 * k] + x
    ls = I._pack(loops, dtype, {}, "thrown", 0)
    want = oracle.aabb_pairs(ls.xyz, ls.offsets)
    xyz, off = torch.from_numpy(ls.xyz).cuda(), torch.from_numpy(ls.offsets).cuda()
    try:
        for method in (0, 1):
            ctx.set_option(lk_mod._lib.OPT_PAIR_SEARCH, method)
            got = ctx.build_pairs(xyz, off).cpu().numpy()
            assert np.array_equal(got, want), method
    finally:
        ctx.set_option(lk_mod._lib.OPT_PAIR_SEARCH, 0)
    print(thrown, centre, dtype.__name__, len(want), "pairs", flush=True)
