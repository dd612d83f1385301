"""The pivot tests of the cluster trees at the edges of a wavefront's tiles: rows of 1 to 8 pieces, the last one
padded, numbers of points around 32, 64 and 128, and leaves so small that the 32 points of a tile belong
to many nodes.  Byte rows are whole numbers: the trees must be the oracle's."""
import numpy as np
import pytest

from helpers import dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,lo,hi", [(np.uint8, 0, 256), (np.int8, -128, 128)])
@pytest.mark.parametrize("d", [7, 32, 100, 128])
def test_trees_equal_the_oracles(env, d, dtype, lo, hi):
    torch, A, O = env
    rng = np.random.default_rng(d)
    pts_h = rng.integers(lo, hi, (4099, d)).astype(dtype)
    pts_h[::5] = pts_h[2]  # equal points: nodes that nothing separates
    for n, Ls in ((31, 2), (33, 2), (65, 3), (129, 2), (513, 4), (2049, 2), (4099, 2), (4099, 700)):
        say(f"cluster tree sides d={d} {dtype.__name__} n={n} Ls={Ls}")
        perm, off, _ = A.ann_hcnng_tree_edges(dev(torch, pts_h[:n]), Ls, 3, 3, 5, 1)
        operm, ooff = O.hcnng_tree(O.Dataset(pts_h[:n], 0), Ls, 5, 1)
        assert (off == ooff[:len(off)]).all() and (perm == operm).all()


def test_allocator_callbacks(env):
    """Graph and scratch come from the caller's callbacks and go back to them, on the default stream and on
    another; an allocator that runs dry gives ANN_ENOMEM and gets everything back."""
    from test_gpu_boundary import CountingAllocator
    torch, A, O = env
    rng = np.random.default_rng(5)
    pts_h = rng.integers(0, 256, (3000, 64)).astype(np.uint8)
    pts = dev(torch, pts_h)
    og = O.hcnng_build(O.Dataset(pts_h, 0), 5, 100, 3, 10, 24, 1.2, seed=3, threads=0)
    for name in (None, "torch"):
        assert (A.ann_hcnng_build(pts, 5, 100, 3, 10, 24, 1.2, seed=3, allocator=name).neighbors() == og).all()
    ca = CountingAllocator(A, torch)
    other = torch.cuda.Stream()
    other.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(other):
        g = A.ann_hcnng_build(pts, 5, 100, 3, 10, 24, 1.2, seed=3, allocator=ca)
    assert (g.neighbors() == og).all() and ca.allocs > 10 and len(ca.live) == 3
    del g
    assert len(ca.live) == 0 and ca.allocs == ca.frees
    for k in (0, 2, 9):
        dry = CountingAllocator(A, torch, fail_after=k)
        with pytest.raises(A.AnnError) as e:
            A.ann_hcnng_build(pts, 5, 100, 3, 10, 24, 1.2, seed=3, allocator=dry)
        assert e.value.code == -2 and len(dry.live) == 0 and dry.allocs == dry.frees == k
