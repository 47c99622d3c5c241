"""Offsets that decrease in a call with few pairs whose preparation scans the
vertices in pieces: such a loop is invalid by itself and every other loop keeps
its own flags.  The flags and integers equal those of the same pairs in a call
with many pairs, which scans a loop per wavefront, and what a loop of the scene
must carry (a bad vertex, no length) is stated here.  Every offset stays inside
the vertex array."""
import numpy as np
import pytest

import paper_2106_12655_amd as lk_mod

pytestmark = pytest.mark.gpu

N, SIZE, FIRST = 48, 1500, 100  # loops, vertices each, vertices before the first


def _scene(seed):
    rng = np.random.default_rng(seed)
    t = 2 * np.pi * np.arange(SIZE) / SIZE
    loops = [np.stack([np.cos(t), np.sin(t), 0.3 * np.sin(2 * t)], 1)
             @ np.linalg.qr(rng.normal(size=(3, 3)))[0] + rng.uniform(-0.7, 0.7, 3) for _ in range(N)]
    xyz = np.concatenate([rng.normal(size=(FIRST, 3))] + loops)
    return xyz, FIRST + SIZE * np.arange(N + 1, dtype=np.int64)


# entry of the offsets -> its value
ENTRIES = {
    "low": {7: 40},                         # before the first loop
    "zero": {5: 0},
    "equal to an earlier": {20: FIRST + 18 * SIZE},
    "high": {9: FIRST + 30 * SIZE + 7},
    "inside a loop": {30: FIRST + 28 * SIZE + 700},
    "two": {3: FIRST + 10, 40: FIRST + 12 * SIZE + 1},
    "last": {N: FIRST + 3 * SIZE},
    "last below the first": {N: 50},
    "first above": {0: FIRST + 2 * SIZE + 5},
}


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("entries", list(ENTRIES))
def test_decreasing_offsets_in_pieces(ctx, entries, dtype):
    import torch
    xyz, off = _scene(len(entries))
    for k, v in ENTRIES[entries].items():
        off[k] = v
    sizes = np.diff(off)
    assert off.min() >= 0 and off.max() <= len(xyz) and sizes.min() < 0
    bad = np.nonzero(sizes < 3)[0]
    good = [l for l in range(N) if sizes[l] == SIZE]
    # loops with a bad vertex or a segment of no length in their later parts (one or
    # the other: a bad vertex leaves no mean coordinate for the length test)
    marked = [good[0], good[len(good) // 2], good[-1]]
    order = np.random.default_rng(1).permutation(good)
    pairs = [(int(a), int(b)) for a, b in zip(order, np.roll(order, 1))]
    pairs += [(int(b), good[1]) for b in bad] + [(good[2], int(b)) for b in bad]
    o = torch.from_numpy(off).cuda()
    print(entries, dtype.__name__, "sizes", sizes.min(), sizes.max(), flush=True)

    def run(x, p):
        out = ctx.direct_sum(x, o, torch.tensor(p, dtype=torch.int32, device="cuda"), mode="mixed")
        torch.cuda.synchronize()
        return [t.cpu().numpy()[:len(pairs)] for t in out]

    # (the length test compares with the mean coordinate of off[-1] - off[0] vertices)
    for plant in ("vertex", "length") if off[-1] > off[0] else ("vertex",):
        y = xyz.copy()
        for k, l in enumerate(marked):
            at = off[l] + SIZE - 5
            y[at] = y[at - 1] if plant == "length" else (np.nan, np.inf, -np.inf)[k]
        x = torch.from_numpy(y.astype(dtype)).cuda()
        # flags of an earlier call in the same workspace: every loop bad
        ctx.direct_sum(torch.full_like(x, float("nan")),
                       torch.linspace(0, len(xyz), N + 1, dtype=torch.float64).long().cuda(),
                       torch.tensor(pairs, dtype=torch.int32, device="cuda"), mode="mixed")
        few = run(x, pairs)
        many = run(x, pairs * (1 + 600 // len(pairs)))
        assert np.array_equal(few[2] & ~1, many[2] & ~1), plant
        assert np.array_equal(few[1], many[1]), plant
        for (a, b), f in zip(pairs, few[2]):
            if a in marked or b in marked or a in bad or b in bad:
                assert f & lk_mod.FLAG_BADLOOP, (plant, a, b, int(f))
            elif sizes[a] == SIZE and sizes[b] == SIZE:
                assert f & ~1 == 0, (plant, a, b, int(f))
