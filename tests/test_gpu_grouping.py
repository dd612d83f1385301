"""Step 2 of a batch at the lines between its forms: how the edges are grouped (by their number and the bits of an
id) and in how many launches the rows are pruned again (by the batch's size and the row's).  Byte rows: graphs
equal the oracle's."""
import numpy as np
import pytest

from helpers import dev, say

pytestmark = pytest.mark.gpu


def _points(n, d, rng):
    c = rng.integers(0, 256, (40, d))
    return np.clip(c[rng.integers(0, 40, n)] + rng.normal(0, 14, (n, d)), 0, 255).astype(np.uint8)


# batches of 1,024 / 1,025, 3,072 / 3,073 and 4,096 / 4,097 points on rows of up to 128 bytes, of 512 / 513, 1,536 / 1,537 and
# 2,560 / 2,561 on wider ones; 1,024, 1,032 and 12,288, 12,320 keys; 10, 11, 12 and 15 bits of an id
@pytest.mark.parametrize("n,d,R,batch", [
    (700, 20, 8, 128), (700, 20, 8, 129), (3000, 32, 16, 768), (3000, 32, 16, 770), (1023, 16, 32, 500), (1025, 16, 32, 500),
    (2049, 128, 24, 1024), (2049, 128, 24, 1025), (17_000, 24, 12, 4096), (17_000, 24, 12, 4097), (3000, 150, 20, 512),
    (3000, 150, 20, 513), (5000, 200, 20, 1280), (5000, 200, 20, 1281), (5000, 200, 20, 1536), (5000, 200, 20, 1537),
    (8000, 136, 12, 2560), (8000, 136, 12, 2561), (14_000, 40, 12, 3072), (14_000, 40, 12, 3073),
    (9000, 180, 100, 2400), (20_000, 64, 64, 20_000)])
def test_batches_equal_the_oracles(env, n, d, R, batch):
    torch, A, O = env
    say(f"grouping n={n} d={d} R={R} batch={batch}")
    pts_h = _points(n, d, np.random.default_rng(n + d))
    want, s = O.build(O.Dataset(pts_h, 0), R, 32, 1.2, seed=2, theta=batch, threads=0)
    g = A.ann_build(dev(torch, pts_h), R, 32, 1.2, seed=2, batch_cap=batch)
    assert g.info().start == s and np.array_equal(g.neighbors(), want)


# thirty thousand edges to one vertex: most of a batch in one bucket, whatever its size
@pytest.mark.parametrize("n", [40_000, 1 << 20])
def test_a_crowded_destination(env, n):
    torch, A, O = env
    say(f"grouping crowded destination n={n}")
    R, d = 16, 16
    rng = np.random.default_rng(4)
    pts_h = rng.integers(0, 256, (n, d)).astype(np.uint8)
    s = n - 1
    g = A.ann_graph_from_host(np.full((n, R), 0xFFFFFFFF, np.uint32), d, A.U8, A.L2SQ, s)
    want = O.empty_graph(n, R)
    ids = rng.permutation(n - 1)[:30_000].astype(np.uint32)
    A.ann_insert_batch(g, dev(torch, pts_h), ids, 32, 1.2)
    O.batch_insert(O.Dataset(pts_h, 0), want, s, ids, 32, 1.2, threads=0)
    assert np.array_equal(g.neighbors(), want)


# every edge of a batch to one vertex, ids of 20, 21 and 22 bits (the last: the radix sort), rows that fill up
@pytest.mark.parametrize("n", [(1 << 20) - 1, 1 << 20, (1 << 21) - 1, 1 << 21])
def test_one_destination(env, n):
    torch, A, O = env
    say(f"grouping one destination n={n}")
    R, d = 16, 16
    rng = np.random.default_rng(3)
    pts_h = rng.integers(0, 256, (n, d)).astype(np.uint8)
    ds = O.Dataset(pts_h, 0)
    pts = dev(torch, pts_h)
    s = n - 1
    g = A.ann_graph_from_host(np.full((n, R), 0xFFFFFFFF, np.uint32), d, A.U8, A.L2SQ, s)
    want = O.empty_graph(n, R)
    for lo in (0, 1000):  # the second batch finds the first's choice of neighbours
        ids = rng.permutation(np.arange(lo, lo + 1000, dtype=np.uint32)) * np.uint32(n // 2003)
        A.ann_insert_batch(g, pts, ids, 32, 1.2)
        O.batch_insert(ds, want, s, ids, 32, 1.2, threads=0)
        assert np.array_equal(g.neighbors(), want)
