"""The persistent kernel's work queues: numbers of items around a round of the
grid and the switch between one queue and several, in small, whole and split
pairs.  Every pair is summed once whatever queue its item came from: a list that
repeats some pairs gives each the same value, bit for bit, wherever it stands."""
import numpy as np
import pytest

import paper_2106_12655_amd as lk_mod
from paper_2106_12655_amd import _lib

pytestmark = pytest.mark.gpu

SIZES = {"small": [30, 64, 100, 127], "whole": [128, 150, 200, 90], "split": [300, 700, 515, 900],
         "mixed": [31, 700, 64, 260, 3, 2000]}


@pytest.mark.parametrize("kind", list(SIZES))
@pytest.mark.parametrize("mode,waves,count", [
    ("mixed", 4, 600), ("mixed", 4, 1023), ("mixed", 4, 1025), ("mixed", 1, 2049),
    ("plain", 2, 4097), ("crossings", 4, 8200), ("mixed", 0, 40001)])
def test_every_item_once(ctx, kind, mode, waves, count):
    import torch
    rng = np.random.default_rng(count)
    sizes = SIZES[kind]
    if count > 9000 and kind in ("split", "mixed"):
        count = 9001
    xyz = np.concatenate([np.stack([np.cos(t), np.sin(t), 0.3 * np.sin(2 * t)], 1)
                          @ np.linalg.qr(rng.normal(size=(3, 3)))[0] + rng.uniform(-0.7, 0.7, 3)
                          for t in (np.arange(n) * 2 * np.pi / n for n in sizes)])
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    distinct = np.array([(i, j) for i in range(len(sizes)) for j in range(len(sizes)) if i != j])
    which = rng.integers(0, len(distinct), count)
    print(kind, mode, waves, count, flush=True)
    ctx.set_option(_lib.OPT_WAVES_PER_CU, waves)
    try:
        out = ctx.direct_sum(torch.from_numpy(xyz).cuda(), torch.from_numpy(off).cuda(),
                             torch.from_numpy(distinct[which].astype(np.int32)).cuda(), mode=mode)
        torch.cuda.synchronize()
    finally:
        ctx.set_option(_lib.OPT_WAVES_PER_CU, 0)
    real, whole, flags = [t.cpu().numpy() for t in out]
    for k in range(len(distinct)):
        got = real[which == k]
        assert len(got) == 0 or np.all(got == got[0]), k
        assert np.abs(got - np.rint(got)).max(initial=0) < 0.05  # no term twice or missing
        assert np.all(whole[which == k] == np.rint(got))
