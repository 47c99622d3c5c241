"""LK_OPT_WAVES_PER_CU holds for the teams of waves that calls with few pairs run
on: lk_get_stats reports at most that many, and the values do not depend on it."""
import numpy as np
import pytest

from paper_2106_12655_amd import _lib
from paper_2106_12655_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["mixed", "plain"])
def test_waves_per_cu_of_few_pairs(ctx, mode):
    import torch
    ls = I.ring_grid(1, rows=6, cols=6, nseg=150)
    x, o = torch.from_numpy(np.ascontiguousarray(ls.xyz)).cuda(), torch.from_numpy(ls.offsets).cuda()
    pairs = ctx.build_pairs(x, o)
    assert len(pairs) <= 512
    values = []
    try:
        for n in (0, 1, 2, 3, 4, 7, 8, 12, 64):
            ctx.set_option(_lib.OPT_WAVES_PER_CU, n)
            out = ctx.direct_sum(x, o, pairs, mode)
            torch.cuda.synchronize()
            used = ctx.stats()["waves_per_cu"]
            print(mode, n, "->", used, flush=True)
            assert used >= 1 and (n == 0 or used <= n)
            values.append([t.cpu().numpy() for t in out])
    finally:
        ctx.set_option(_lib.OPT_WAVES_PER_CU, 0)
    for v in values[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(v, values[0]))
