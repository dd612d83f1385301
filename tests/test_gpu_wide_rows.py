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


@pytest.mark.parametrize("d,R", [(80, 128), (80, 129), (112, 150), (96, 150), (144, 150), (256, 200), (272, 130)])
def test_many_edges_per_vertex(env, d, R):
    """Each walk of the prune where R is long: copies of the selected rows that fill their LDS or no longer fit it
    (rows of 80 and 112 bytes on both sides of R = 128), rows read from device memory, rows above 256 bytes."""
    torch, A, O = env
    rng = np.random.default_rng(d + R)
    pts_h = rng.integers(0, 256, (1200, d)).astype(np.uint8)  # (nothing clusters: few candidates are removed)
    say(f"many edges d={d} R={R}")
    og, start = O.build(O.Dataset(pts_h, 0), R, 220, 1.0, seed=3, threads=0)
    g = A.ann_build(dev(torch, pts_h), R, 220, 1.0, seed=3)
    assert int(g.info().start) == start and (g.neighbors() == og).all()
    assert ((og != 0xFFFFFFFF).sum(1) > 32).any()
