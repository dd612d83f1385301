"""The search kernel that requests the next hops' memory ahead, at the edges of its range: every result
must be the oracle's, and that of the kernel that takes larger launches."""
import numpy as np
import pytest

from helpers import dev, say

pytestmark = pytest.mark.gpu

KINDS = {"u8": (np.uint8, 128), "u8short": (np.uint8, 60), "i8": (np.int8, 100), "u8wide": (np.uint8, 256), "i8long": (np.int8, 400)}


def _points(kind, n, seed):
    dtype, d = KINDS[kind]
    rng = np.random.default_rng(seed)
    c = rng.standard_normal((40, d)) * 40
    x = c[rng.integers(0, 40, n)] + 20 * rng.standard_normal((n, d))
    x = np.clip(np.round(np.abs(x)), 0, 255) if dtype is np.uint8 else np.clip(np.round(x), -127, 127)
    x = x.astype(dtype)
    x[-60:] = x[:60]  # equal points: ties by id
    return x


@pytest.mark.parametrize("kind,R", [("u8", 64), ("u8", 32), ("u8short", 33), ("i8", 48), ("u8wide", 64), ("i8long", 40)])
def test_requests_ahead_do_not_show(env, kind, R):
    torch, A, O = env
    pts_h, qs_h = _points(kind, 2500, 1), _points(kind, 3100, 2)
    ds = O.Dataset(pts_h, 0)
    pts, qs = dev(torch, pts_h), dev(torch, qs_h)
    g = A.ann_build(pts, R, 64, 1.2, seed=4)
    rows, start = g.neighbors(), int(g.info().start)
    for L in (32, 33, 64, 65, 128):
        for k, eps in ((10, -1.0), (L, 0.0), (1, 0.1)):
            say(f"ahead {kind} R={R} L={L} k={k} eps={eps}")
            ids, dists = A.ann_search_eps(g, pts, qs, k, L, eps)  # (more than this kernel takes)
            for nq in (513, 2048):
                i, d = A.ann_search_eps(g, pts, qs[:nq], k, L, eps)
                assert torch.equal(i, ids[:nq]) and torch.equal(d, dists[:nq])
            oi, od = O.search_batch(ds, rows, start, qs_h[:513], k, L, eps=eps, threads=0)
            assert (i[:513].cpu().numpy().view(np.uint32) == oi).all() and (d[:513].cpu().numpy() == od).all()


def test_requests_ahead_visited_lists(env):
    """Build searches: visited lists are written 64 entries at a time, in their slot, across its end into a
    spill chunk, or are redone where there is no room."""
    torch, A, O = env
    pts_h = _points("u8", 4000, 3)
    pts = dev(torch, pts_h)
    og, _ = O.build(O.Dataset(pts_h, 0), 32, 70, 1.2, seed=2, theta=900, threads=0)
    for kw in ({}, {"visited_cap": 64}, {"visited_cap": 100, "spill_cap": 10 ** 6}, {"visited_cap": 8, "spill_cap": 1}):
        say(f"ahead build {kw}")
        g = A.ann_build(pts, 32, 70, 1.2, seed=2, batch_cap=900, **kw)
        assert (g.neighbors() == og).all()


def test_requests_ahead_start_vertices(env):
    """Searches with start vertices of their own (the layered index)."""
    torch, A, O = env
    pts_h, qs_h = _points("i8", 4000, 5), _points("i8", 600, 6)
    pts, qs = dev(torch, pts_h), dev(torch, qs_h)
    h = A.ann_hnsw_build(pts, 16, 48, 1.2, seed=2, batch_cap=800)
    ds = O.Dataset(pts_h, 0)
    oh = O.hnsw_build(ds, 16, 48, 1.2, seed=2, theta=800, threads=0)
    for l in range(oh.top + 1):
        lid, lrows = h.layer(l)
        assert (lrows == oh.layers[l][lid]).all()
    ids, _ = A.ann_hnsw_search(h, pts, qs, 10, 40)
    assert (ids.cpu().numpy().view(np.uint32) == O.hnsw_search_batch(ds, oh, qs_h, 10, 40, threads=0)[0]).all()


@pytest.mark.parametrize("n", [(1 << 20) + 1, (1 << 22) + 1])
def test_requests_ahead_many_points(env, n):
    """Ids of 21 and 23 bits, the most that 16-bit tags hold in the filters of this kernel and of the one for
    larger launches."""
    torch, A, _ = env
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    c = torch.randint(256, (3000, 16), generator=g, device="cuda")

    def rows(m):
        x = c[torch.randint(3000, (m,), generator=g, device="cuda")] + torch.randint(-40, 41, (m, 16), generator=g, device="cuda")
        return x.clamp_(0, 255).to(torch.uint8)

    pts, qs = rows(n), rows(3100)
    graph = A.ann_build(pts, 32, 48, 1.2, seed=6)
    for L in (32, 64, 128):
        say(f"ahead n={n} L={L}")
        ids, dists = A.ann_search(graph, pts, qs, 10, L)
        i, d = A.ann_search(graph, pts, qs[:3000], 10, L)
        assert torch.equal(i, ids[:3000]) and torch.equal(d, dists[:3000])
