"""A leaf's pair sort and tree scan where they can go wrong: leaves of every size class (up to 4,096, 8,192 and 16,384
pairs), one entry per list up to sixteen, distances that crowd into one bucket (equal points, few
distinct values), a far point that stretches the span, trees whose points fill up (s = 1).  The accepted pairs are
the oracle's, in its order."""
import numpy as np
import pytest

from helpers import dev, say

pytestmark = pytest.mark.gpu


def _points(kind, n, d, rng):
    x = rng.integers(0, 256, (n, d)).astype(np.uint8)
    if kind == "equal":
        x[:] = x[0]
    elif kind == "few":  # distances take a handful of values
        x = rng.integers(0, 2, (n, d)).astype(np.uint8)
    elif kind == "far":  # one dense cloud, one point far away
        x = (100 + rng.integers(0, 3, (n, d))).astype(np.uint8)
        x[n // 2] = 255
    elif kind == "half":  # every other point the same one
        x[::2] = x[1]
    return x


@pytest.mark.parametrize("kind", ["spread", "equal", "few", "far", "half"])
def test_leaves_equal_the_oracles(env, kind):
    torch, A, O = env
    for n, l, s, d in ((2, 3, 3, 8), (3, 1, 1, 8), (64, 10, 3, 16), (65, 16, 2, 16), (409, 10, 3, 32), (410, 10, 3, 32),
                       (819, 10, 255, 20), (820, 10, 1, 20), (1024, 1, 3, 8), (1024, 4, 3, 64), (1023, 15, 3, 128), (1024, 16, 3, 128)):
        say(f"cluster pairs {kind} n={n} l={l} s={s}")
        x = _points(kind, n, d, np.random.default_rng(n + l))
        _, off, edges = A.ann_hcnng_tree_edges(dev(torch, x), 1024, s, l, 5, 0)
        want = O.hcnng_leaf(O.Dataset(x, 0), np.arange(n), s, l)
        assert len(off) == 2 and np.array_equal(np.asarray(edges), np.asarray(want)), (n, l, s)


@pytest.mark.parametrize("n,T,s,Ls,dtype", [(64, 32, 3, 20, "u8"), (65, 24, 4, 30, "u8"), (700, 33, 3, 50, "u8"), (700, 25, 4, 64, "u8"),
                                            (701, 3, 5, 60, "u8"), (127, 96, 1, 9, "u8"), (640, 1, 2, 33, "u8"), (2, 4, 3, 5, "u8"),
                                            (700, 32, 3, 50, "f32"), (300, 40, 3, 50, "f32")])
def test_neighbours_of_all_trees(env, n, T, s, Ls, dtype):
    """Trees times s at 96 and beyond, s at 4 and beyond, points around a workgroup's 64: graphs equal the oracle's."""
    torch, A, O = env
    say(f"cluster collect n={n} T={T} s={s}")
    rng = np.random.default_rng(n + T)
    x = rng.integers(0, 256, (n, 32)).astype(np.uint8)
    if dtype == "f32":  # whole numbers: the distances are exact in fp32
        x = x.astype(np.float32)
    g = A.ann_hcnng_build(dev(torch, x), T, Ls, s, 10, 24, 1.2, seed=3)
    assert np.array_equal(g.neighbors(), O.hcnng_build(O.Dataset(x, 0), T, Ls, s, 10, 24, 1.2, seed=3, threads=0))


def test_order_across_spans(env):
    """Two of 512 pairs share a point that takes one neighbour.  Their distances lie on both sides of the line between two
    spans of the pair sort, three units in the last place apart, such that the larger one's product with the scale is
    less than a whole number by less than its rounding, in a span that 261 pairs share, right behind one that the smaller one has
    for itself (pairs that lie far apart from all others; their first coordinate keeps them so)."""
    torch, A, O = env
    f = np.float32
    close = [f(1.1101452112197876), f(1.1101453304290771)]  # the first wins
    span = int(np.frombuffer(f(929955008.0 * 929955008.0).tobytes(), np.uint32)[0] - 0x3F800000) / 1024
    at = [span * 0.999 * i / 249 for i in range(249)] + [span * (4.001 + 0.99 * i / 260) for i in range(260)]
    alone = [f(np.sqrt(np.frombuffer(np.uint32(0x3F800000 + int(k)).tobytes(), f)[0])) for k in at] + [f(929955008.0)]
    rows = [(0.0, -close[0]), (0.0, 0.0), (0.0, close[1])]
    for i, gap in enumerate(alone):
        rows += [((i + 1) * 2.0 ** 40, 0.0), ((i + 1) * 2.0 ** 40, gap)]
    x = np.zeros((len(rows), 4), f)
    x[:, :2] = rows
    _, off, edges = A.ann_hcnng_tree_edges(dev(torch, x), 1024, 1, 1, 5, 0)
    want = O.hcnng_leaf(O.Dataset(x, 0), np.arange(len(x)), 1, 1)
    assert len(off) == 2 and len(want) == 511
    assert np.array_equal(np.asarray(edges), np.asarray(want))
