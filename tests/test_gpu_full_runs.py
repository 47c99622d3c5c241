"""The direct sum where all angles are large: polygons of random vertices, whose
walks go over to runs of 64 steps that take the full arctangent without a test.
Loop lengths stand around the ends of such runs (four tested steps, then up to
64) and of what follows them; smooth loops share waves with them.

Every form gives the same value, so a pair's value must not depend, in any bit,
on what shares its wave, nor (for pairs of big items) on the kernel that ran it.
Integers equal the oracle's; FP64 values lie within 1e-9 of it (at most 5e5 terms
of relative error below 1e-15 each, and closest segments some 1e-5 apart)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SIZES = [3, 4, 5, 7, 8, 9, 67, 68, 69, 71, 72, 73, 75, 76, 127, 128, 135, 136, 137, 140, 205, 300, 700]


def _scene(dtype):
    rng = np.random.default_rng(11)
    loops = [rng.normal(size=(n, 3)) for n in SIZES]
    for n in (40, 64, 120, 500):  # small angles
        t = 2 * np.pi * np.arange(n) / n
        loops.append(np.stack([6 * np.cos(t), 6 * np.sin(t), np.sin(2 * t)], 1))
    xyz = np.concatenate(loops).astype(dtype)
    off = np.concatenate([[0], np.cumsum([len(x) for x in loops])]).astype(np.int64)
    # (the smooth loops follow one curve: not with each other)
    i, j = np.nonzero(~np.eye(len(loops), dtype=bool))
    i, j = i[np.minimum(i, j) < len(SIZES)], j[np.minimum(i, j) < len(SIZES)]
    return xyz, off, np.stack([i, j], 1).astype(np.int32)


@pytest.mark.parametrize("mode", ["mixed", "plain"])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_runs_of_large_angles(ctx, dtype, mode):
    import torch
    xyz, off, pairs = _scene(dtype)
    x, o = torch.from_numpy(xyz).cuda(), torch.from_numpy(off).cuda()
    want, ints = oracle.direct_sum(xyz, off, pairs)

    def run(order):
        out = ctx.direct_sum(x, o, torch.from_numpy(pairs[order]).cuda(), mode)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in out]

    n = len(pairs)
    assert n > 512  # items on single waves
    real, lk, flags = run(np.arange(n))
    order = np.random.default_rng(2).permutation(n)
    back = np.empty(n)
    back[order] = run(order)[0]
    err = np.abs(real - want).max()
    print("%s %s: %d pairs, %d refits, max |err| %.1e" % (
        np.dtype(dtype).name, mode, n, int((flags & 1).sum()), err), flush=True)
    assert np.array_equal(lk, ints) and np.all(flags & ~1 == 0)
    assert np.array_equal(real, back)
    assert mode == "mixed" or err <= 1e-9
    few = run(order[:400])  # teams of waves
    sizes = np.diff(off)
    big = sizes[pairs[order[:400], 0]] >= 128
    assert np.array_equal(few[0][big], real[order[:400]][big])
    assert np.array_equal(few[1], ints[order[:400]])
