"""Float rows at the edges of the kernels' instances (pieces per lane: up to 128 elements 2 or 4, up to
192 six, up to 224 seven, up to 256 eight; full last pieces and partly empty ones).  The elements are
small whole numbers: every sum is exact in fp32 whatever its order, so that graphs, ids and
distances must be the oracle's bit for bit."""
import numpy as np
import pytest

from helpers import dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("metric,alpha", [(0, 1.2), (1, 1.0)])
@pytest.mark.parametrize("d", [64, 68, 128, 132, 160, 192, 196, 224, 228, 256])
def test_whole_numbers_bit_exact(env, d, metric, alpha):
    torch, A, O = env
    rng = np.random.default_rng(d)
    c = rng.integers(-6, 7, (30, d))

    def rows(n):
        return (c[rng.integers(0, 30, n)] + rng.integers(-3, 4, (n, d))).astype(np.float32)

    pts_h, qs_h = rows(1500), rows(1100)
    ds, pts, qs = O.Dataset(pts_h, metric), dev(torch, pts_h), dev(torch, qs_h)
    for R, L in ((8, 24), (48, 70)):  # selected rows that the prune stages in LDS, and that it cannot
        say(f"float rows d={d} metric={metric} build R={R}")
        og, start = O.build(ds, R, L, alpha, seed=3, threads=0)
        g = A.ann_build(pts, R, L, alpha, seed=3, metric=metric)
        assert int(g.info().start) == start and (g.neighbors() == og).all()
    for Ls, eps in ((20, -1.0), (64, -1.0), (100, -1.0), (200, -1.0), (100, 0.1)):
        oi, od = O.search_batch(ds, og, start, qs_h, 10, Ls, eps=eps, threads=0)
        for nq in (37, 1100):  # several waves per search, one
            say(f"float rows d={d} metric={metric} L={Ls} eps={eps} nq={nq}")
            ids, dists = A.ann_search_eps(g, pts, qs[:nq], 10, Ls, eps)
            assert (ids.cpu().numpy().view(np.uint32) == oi[:nq]).all() and (dists.cpu().numpy() == od[:nq]).all()
    say(f"float rows d={d} metric={metric} layers")
    oh = O.hnsw_build(ds, 16, 40, alpha, seed=5, threads=0)
    h = A.ann_hnsw_build(pts, 16, 40, alpha, seed=5, metric=metric)
    for Ls in (12, 64):
        ids, dists = A.ann_hnsw_search(h, pts, qs, 10, Ls)
        oi, od, _ = O.hnsw_search_batch(ds, oh, qs_h, 10, Ls, threads=0)
        assert (ids.cpu().numpy().view(np.uint32) == oi).all() and (dists.cpu().numpy() == od).all()
