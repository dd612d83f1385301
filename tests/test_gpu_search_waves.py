"""The search kernel that shares a search between several waves, at the edges of its range: every
result must be that of the one-wave kernel (whole batches of more than 1,024 queries) and, for
integer rows, of the oracle."""
import numpy as np
import pytest

from helpers import dev, say

pytestmark = pytest.mark.gpu

KINDS = {"u8": (np.uint8, 0, 128), "i8": (np.int8, 0, 100), "f32": (np.float32, 0, 48), "f32ip": (np.float32, 1, 200),
         "u8wide": (np.uint8, 0, 256)}


def _points(kind, n, seed):
    dtype, metric, d = KINDS[kind]
    rng = np.random.default_rng(seed)
    c = rng.standard_normal((40, d)) * 40
    x = c[rng.integers(0, 40, n)] + 20 * rng.standard_normal((n, d))
    if dtype is np.uint8:
        x = np.clip(np.round(np.abs(x)), 0, 255)
    elif dtype is np.int8:
        x = np.clip(np.round(x), -127, 127)
    else:
        x = x / np.linalg.norm(x, axis=1, keepdims=True)
    x = x.astype(dtype)
    x[-60:] = x[:60]  # equal points: ties by id
    return x


@pytest.mark.parametrize("kind,R,Lb", [("u8", 64, 64), ("i8", 33, 40), ("f32", 32, 64), ("f32ip", 64, 64), ("u8wide", 1, 32)])
def test_waves_per_search_do_not_show(env, kind, R, Lb):
    torch, A, O = env
    dtype, metric, d = KINDS[kind]
    pts_h, qs_h = _points(kind, 2500, 1), _points(kind, 1100, 2)
    ds = O.Dataset(pts_h, metric)
    pts, qs = dev(torch, pts_h), dev(torch, qs_h)
    g = A.ann_build(pts, R, Lb, 1.0 if metric else 1.2, seed=4, metric=metric)
    rows, start = g.neighbors(), int(g.info().start)
    cuts = [0, 1, 38, 550, 1100]  # 1, 37, 512 queries: eight waves; 550: one, the graph is small
    for L in (31, 32, 64, 65, 128, 129, 256):
        for k, eps in ((10, -1.0), (L, -1.0), (10, 0.0), (10, 0.1)):
            say(f"waves {kind} L={L} k={k} eps={eps}")
            ids, dists = A.ann_search_eps(g, pts, qs, k, L, eps)
            part = [A.ann_search_eps(g, pts, qs[a:b], k, L, eps) for a, b in zip(cuts, cuts[1:])]
            assert torch.equal(torch.cat([p[0] for p in part]), ids)
            assert torch.equal(torch.cat([p[1] for p in part]), dists)
            if dtype is not np.float32:
                oi, od = O.search_batch(ds, rows, start, qs_h, k, L, eps=eps, threads=0)
                assert (ids.cpu().numpy().view(np.uint32) == oi).all() and (dists.cpu().numpy() == od).all()


def test_waves_per_search_visited_lists(env):
    """Build searches shared by several waves: visited lists that outgrow their slot move to spill
    chunks, or are redone where there is no room."""
    torch, A, O = env
    pts_h = _points("u8", 2500, 3)
    og, _ = O.build(O.Dataset(pts_h, 0), 24, 48, 1.2, seed=2, threads=0)
    pts = dev(torch, pts_h)
    for kw in ({}, {"visited_cap": 8, "spill_cap": 10 ** 6}, {"visited_cap": 8, "spill_cap": 1}, {"batch_cap": 1030}):
        say(f"waves build {kw}")
        g = A.ann_build(pts, 24, 48, 1.2, seed=2, **kw)
        if "batch_cap" in kw:
            og, _ = O.build(O.Dataset(pts_h, 0), 24, 48, 1.2, seed=2, theta=kw["batch_cap"], threads=0)
        assert (g.neighbors() == og).all()


def test_four_waves_per_search(env):
    """Between 512 and 1,024 searches of a graph beyond the last-level cache share four waves."""
    torch, A, _ = env
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    c = 40 * torch.randn((300, 128), generator=g, device="cuda")

    def rows(n):
        x = c[torch.randint(300, (n,), generator=g, device="cuda")]
        return (x + 25 * torch.randn((n, 128), generator=g, device="cuda")).round_().clamp_(-127, 127).to(torch.int8)

    n = (256 << 20) // (128 + 4 * 64) + 1  # the smallest such graph
    pts, qs = rows(n), rows(1025)
    graph = A.ann_build(pts, 64, 64, 1.2, seed=6)
    for L in (32, 64, 65, 129, 256):
        for eps in (-1.0, 0.1):
            say(f"four waves L={L} eps={eps}")
            ids, dists = A.ann_search_eps(graph, pts, qs, 10, L, eps)
            for nq in (513, 1024):
                i, d = A.ann_search_eps(graph, pts, qs[:nq], 10, L, eps)
                assert torch.equal(i, ids[:nq]) and torch.equal(d, dists[:nq])


@pytest.mark.parametrize("n", [(1 << 20) + 1, (1 << 22) + 1, (1 << 23) + 1])
def test_waves_per_search_many_points(env, n):
    """Ids of 21, 23 and 24 bits: the several-waves kernel's filter keeps 16-bit tags, the one-wave kernel's
    smaller one does not for the last graph."""
    torch, A, _ = env
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    c = torch.randint(256, (3000, 16), generator=g, device="cuda")

    def rows(m):
        x = c[torch.randint(3000, (m,), generator=g, device="cuda")] + torch.randint(-40, 41, (m, 16), generator=g, device="cuda")
        return x.clamp_(0, 255).to(torch.uint8)

    pts, qs = rows(n), rows(1100)
    graph = A.ann_build(pts, 48, 48, 1.2, seed=6)
    for L in (32, 64, 128, 256):
        say(f"several waves n={n} L={L}")
        ids, dists = A.ann_search(graph, pts, qs, 10, L)
        for nq in (1, 37, 512, 1000):
            i, d = A.ann_search(graph, pts, qs[:nq], 10, L)
            assert torch.equal(i, ids[:nq]) and torch.equal(d, dists[:nq])
