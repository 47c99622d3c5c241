"""The pair search at the number of loops from which the rows' places come from a
scanned list of tile sums: lattices of small boxes with a known list of pairs, and
a buffer that is one pair too small."""
import ctypes

import numpy as np
import pytest

import paper_2106_12655_amd as lk_mod

pytestmark = pytest.mark.gpu

TILES = 1024 * 256


@pytest.mark.parametrize("n", [TILES - 1, TILES, TILES + 1, TILES + 256, 2 * TILES + 77])
def test_lattice_of_triangles(ctx, n):
    import torch
    # boxes of side 0.6 at (k mod w, k div w) / 2: each meets the next in its row and in
    # its column, and those across the corner
    w = 701
    k = torch.arange(n, device="cuda")
    lo = torch.stack([k % w, k // w, torch.zeros_like(k)], 1).float() * 0.5
    tri = torch.tensor([[0, 0, 0], [0.6, 0.3, 0.1], [0.3, 0.6, 0.6]], device="cuda")
    xyz = (lo[:, None] + tri).reshape(-1, 3).contiguous()
    off = torch.arange(n + 1, device="cuda") * 3
    parts = []
    for d, ok in ((1, k % w < w - 1), (w - 1, k % w > 0), (w, k >= 0), (w + 1, k % w < w - 1)):
        i = k[ok & (k + d < n)]
        parts.append(torch.stack([i, i + d], 1))
    want = torch.cat(parts)
    want = want[torch.argsort(want[:, 0] * n + want[:, 1])].int()
    got = ctx.build_pairs(xyz, off)
    print("%d loops: %d pairs" % (n, len(want)), flush=True)
    assert torch.equal(got, want)
    out = torch.full((len(want), 2), -7, dtype=torch.int32, device="cuda")
    cnt = ctypes.c_int64(0)
    st = ctx.lib.lk_build_pairs(ctx.h, xyz.data_ptr(), 0, off.data_ptr(), n, out.data_ptr(),
                                len(want) - 1, ctypes.byref(cnt), None)
    assert st == lk_mod._lib.ECAPACITY and cnt.value == len(want) and bool((out == -7).all())
