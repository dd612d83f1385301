"""The prune and re-prune of float rows on the matrix cores, where their blocks of 16 candidates and tiles of 16
rows begin and end, where a list passes 128 entries, and where their products cannot decide a pair.  Elements are small whole numbers times a
power of two (or moved far from the origin): every sum is exact in fp32, so that graphs must be the
oracle's bit for bit; ties between distances, which only a measured distance settles, are common.
Scaled by 2^-70, squares and their sums are subnormal."""
import numpy as np
import pytest

from helpers import dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("metric,alpha", [(0, 1.2), (0, 1.0), (1, 1.0)])
@pytest.mark.parametrize("d,offset,scale", [(4, 0, 1.0), (28, 4096, 1.0), (60, 0, 2.0 ** -70), (132, 0, 2.0 ** 40), (256, 512, 1.0)])
def test_blocks_and_ties(env, d, offset, scale, metric, alpha):
    torch, A, O = env
    if metric == 1 and offset:
        offset = 8  # (inner products of far rows would not be exact)
    rng = np.random.default_rng(1000 * metric + d)
    c = rng.integers(-3, 4, (12, d))
    base = (c[rng.integers(0, 12, 700)] + rng.integers(-1, 2, (700, d)) + offset).astype(np.float32)
    base[::7] = base[3]  # (a point many times over)
    pts_h = base * np.float32(scale)
    for n, R, L in ((17, 16, 20), (33, 15, 16), (700, 17, 33), (700, 33, 90), (700, 64, 128), (700, 110, 128)):
        say(f"float prune d={d} offset={offset} scale={scale} metric={metric} alpha={alpha} n={n} R={R}")
        og, start = O.build(O.Dataset(pts_h[:n], metric), R, L, alpha, seed=3, threads=0)
        g = A.ann_build(dev(torch, pts_h[:n]), R, L, alpha, seed=3, metric=metric)
        assert int(g.info().start) == start and (g.neighbors() == og).all()
