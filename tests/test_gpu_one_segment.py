"""One segment of loop B per lane: a call with few pairs takes the arctangent of the
full range alone, one with many the short forms too.  A pair's value is the same to
the last bit in both (with one segment per lane nothing is packed), and integers
equal the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2106_12655_amd import _lib
from paper_2106_12655_amd import inputs as I

pytestmark = pytest.mark.gpu

SIZES = [3, 5, 63, 64, 65, 126, 127, 128, 129, 200, 257, 513, 1025, 2050]


@pytest.mark.parametrize("form", [0, 1, 2])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_few_and_many_pairs_agree(ctx, dtype, form):
    import torch
    rng = np.random.default_rng(4)
    loops = [np.stack([np.cos(t), np.sin(t), 0.3 * np.sin(2 * t)], 1) @ I.random_rotation(rng).T
             + rng.uniform(-0.7, 0.7, 3) for n in SIZES for t in [2 * np.pi * np.arange(n) / n]]
    xyz = np.concatenate(loops).astype(dtype)
    off = np.concatenate([[0], np.cumsum(SIZES)]).astype(np.int64)
    i, j = np.nonzero(~np.eye(len(SIZES), dtype=bool))
    pairs = np.stack([i, j], 1).astype(np.int32)
    x, o = torch.from_numpy(xyz).cuda(), torch.from_numpy(off).cuda()

    def run(p):
        out = ctx.direct_sum(x, o, torch.from_numpy(p).cuda(), "mixed")
        torch.cuda.synchronize()
        return [t.cpu().numpy()[:len(pairs)] for t in out]

    options = {_lib.OPT_SEGS_PER_LANE: 1, _lib.OPT_SEGS_PER_LANE_F64: 1, _lib.OPT_ATAN: form}
    try:
        for k, v in options.items():
            ctx.set_option(k, v)
        few, many = run(pairs), run(np.concatenate([pairs] * 5))
    finally:
        for k in options:
            ctx.set_option(k, 0)
    print(dtype.__name__, "form", form, len(pairs), "pairs", flush=True)
    for a, b in zip(few, many):
        assert np.array_equal(a, b)
    assert np.array_equal(few[1], oracle.direct_sum(xyz, off, pairs)[1])
