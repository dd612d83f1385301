"""Byte rows of 129 to 256 bytes: the matrix-core prune and re-prune with eight k-steps.  Row sizes around the
16-byte pieces and 32-byte steps (the last step half empty, or the rows padded), values at the ends of
their range, rows of the graph around the 16, 32 and 64 entries of a block."""
import numpy as np
import pytest

from helpers import dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,lo,hi", [(np.uint8, 0, 255), (np.int8, -128, 127)])
@pytest.mark.parametrize("d", [129, 144, 160, 176, 200, 256])
def test_graphs_equal_the_oracles(env, d, dtype, lo, hi):
    torch, A, O = env
    rng = np.random.default_rng(d)
    c = rng.integers(lo, hi + 1, (25, d))
    pts_h = np.clip(c[rng.integers(0, 25, 1500)] + rng.integers(-30, 31, (1500, d)), lo, hi).astype(dtype)
    pts_h[:40] = np.where(rng.integers(0, 2, (40, d)) == 1, hi, lo)  # the largest distances
    pts_h[::50] = pts_h[1]
    for n, R, L, alpha in ((40, 8, 12, 1.0), (1500, 15, 30, 1.2), (1500, 33, 70, 1.2), (1500, 64, 128, 1.2), (1500, 100, 128, 1.0)):
        say(f"wide rows d={d} {dtype.__name__} n={n} R={R}")
        og, start = O.build(O.Dataset(pts_h[:n], 0), R, L, alpha, seed=3, threads=0)
        g = A.ann_build(dev(torch, pts_h[:n]), R, L, alpha, seed=3)
        assert int(g.info().start) == start and (g.neighbors() == og).all()
