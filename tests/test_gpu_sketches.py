"""Searches over sketches of float rows: graphs and results are those of searches without them, bit for bit."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _points(torch, n, d, kind, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    c = torch.randn((256, d), generator=g, device="cuda")
    x = c[torch.randint(256, (n,), generator=g, device="cuda")] + 0.4 * torch.randn((n, d), generator=g, device="cuda")
    if kind == "far":  # a cloud far from the origin: the bounds are wide against the distances
        x += 30.0
    elif kind == "unit":
        x /= x.norm(dim=1, keepdim=True)
    elif kind == "odd":  # rows that no bound covers, and rows that the rounding serves badly
        s = 7919
        x[0::s] = 0.0
        x[1::s] *= 1e13
        x[2::s] *= 1e-13
        x[3::s, 0] = 50.0
        x[4::s, d - 1] = float("inf")
        x[5::s] = x[7:8]
        x[6::s] *= 3e-39
    return x


class _Refusing:
    """An allocator that has no memory for one size (that of the sketches: no array of rows may have it)."""

    def __init__(self, A, nbytes):
        self.inner = A.TorchAllocator()
        self.refused = 0

        def alloc(size, stream, user):
            if size == nbytes:
                self.refused += 1
                return None
            return self.inner.alloc(size, stream, user)

        self.alloc = A.ALLOC_FN(alloc)
        self.free = self.inner.free

    def fill(self, opts):
        opts.alloc = C.cast(self.alloc, C.c_void_p)
        opts.free = C.cast(self.free, C.c_void_p)
        opts.alloc_user = None


# both sizes of a sketch; 20, 25, 31 (no piece to spare beside the scale), 40, 48, 49, 56, 57 and 63 pieces of 16 bytes;
# one and two slots of the beam, the sorting network
@pytest.mark.parametrize("d,metric,kind,R,L", [
    (80, "l2", "far", 48, 20), (100, "ip", "unit", 64, 64), (124, "l2", "odd", 48, 96), (160, "ip", "odd", 32, 128),
    (192, "l2", "unit", 48, 32), (196, "ip", "far", 48, 65), (224, "l2", "odd", 40, 128), (228, "ip", "unit", 32, 48),
    (252, "l2", "far", 48, 100)])
def test_sketches_change_nothing(env, d, metric, kind, R, L):
    torch, A, _ = env
    sk = 128 if d < 128 else 256
    n = (272 << 20) // (4 * d)
    x = _points(torch, n, d, kind, d)
    m = A.L2SQ if metric == "l2" else A.MIPS
    refusing = _Refusing(A, n * sk)
    kw = dict(seed=3, metric=m, batch_cap=20_000, max_rounds=16)
    g = A.ann_build(x, R, L, 1.0, **kw)
    h = A.ann_build(x, R, L, 1.0, allocator=refusing, **kw)
    assert refusing.refused == 1
    assert np.array_equal(g.neighbors(), h.neighbors()) and g.info().start == h.info().start
    q = _points(torch, 20_001, d, "odd" if kind == "odd" else "unit" if metric == "ip" else kind, d + 1)
    for eps in (-1.0, 0.1):
        a = A.ann_search_eps(g, x, q, 10, L, eps)
        b = A.ann_search_eps(h, x, q, 10, L, eps)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1].view(torch.int32), b[1].view(torch.int32))
    assert refusing.refused == 3


def test_streamed_and_layered(env):
    torch, A, _ = env
    n, d = 345_000, 200
    x = _points(torch, n, d, "unit", 5)
    out = []
    for refuse in (False, True):
        al = _Refusing(A, n * 256) if refuse else "torch"
        g = A.ann_build(x[:300_000], 32, 64, 1.0, seed=2, metric=A.MIPS, allocator=al)
        A.ann_insert_points(g, x, 64, 1.0, seed=4)
        h = A.ann_hnsw_build(x, 16, 64, 1.0, seed=6, metric=A.MIPS, allocator=al)
        r = A.ann_hnsw_search(h, x, x[:30_000], 10, 40)
        out.append((g.neighbors(), h.layer(0)[1], r[0].cpu().numpy(), r[1].cpu().numpy()))
        if refuse:
            assert al.refused == 3  # the insertion, the layered build, the queries on it
    for a, b in zip(*out):
        assert np.array_equal(a, b)


def test_captured_queries_do_without(env):
    """A call under capture neither allocates nor leaves memory of the graph's in what it captured."""
    torch, A, _ = env
    n, d = 350_000, 200
    x = _points(torch, n, d, "unit", 8)
    g = A.ann_build(x, 32, 32, 1.0, seed=2, metric=A.MIPS, batch_cap=20_000, max_rounds=16)
    q = x[:20_000].contiguous()
    want = A.ann_search(g, x, q, 10, 32)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = A.ann_search(g, x, q, 10, 32)
    for _ in range(3):
        got[0].zero_()
        got[1].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_sketch_memory_goes_back(env):
    """What a query call took for sketches is the graph's until it grows or is freed, and then goes back."""
    from test_gpu_boundary import CountingAllocator
    torch, A, _ = env
    n, d = 345_000, 200
    x = _points(torch, n, d, "unit", 5)
    q = x[:20_000].contiguous()
    kw = dict(seed=2, metric=A.MIPS, batch_cap=20_000, max_rounds=16)

    al = CountingAllocator(A, torch)
    g = A.ann_build(x, 32, 32, 1.0, allocator=al, **kw)
    built = len(al.live)
    A.ann_search(g, x, q, 10, 32)
    A.ann_search(g, x, q, 10, 32)
    assert len(al.live) == built + 1
    torch.cuda.synchronize()
    del g
    assert len(al.live) == 0 and al.allocs == al.frees

    al = CountingAllocator(A, torch)
    g = A.ann_build(x[:340_000], 32, 32, 1.0, allocator=al, **kw)
    A.ann_search(g, x[:340_000], q, 10, 32)
    A.ann_insert_points(g, x, 32, 1.0, seed=4)
    A.ann_search(g, x, q, 10, 32)
    torch.cuda.synchronize()
    del g
    assert len(al.live) == 0 and al.allocs == al.frees

    al = CountingAllocator(A, torch)
    h = A.ann_hnsw_build(x, 16, 32, 1.0, allocator=al, **kw)
    built = len(al.live)
    A.ann_hnsw_search(h, x, q, 10, 32)
    assert len(al.live) == built + 2  # the sketches, the queries' start vertices
    torch.cuda.synchronize()
    del h
    assert len(al.live) == 0 and al.allocs == al.frees


def test_queries_do_not_wait(env):
    """A query call returns while its stream is busy, the first one and the first one after an insertion too; its
    sketches stand behind the late work of their memory's last owner, also for a call on another stream."""
    from test_gpu_boundary import CountingAllocator
    torch, A, _ = env
    n, d = 345_000, 200
    x = _points(torch, n, d, "unit", 5)
    q = x[:20_000].contiguous()
    old = x[:340_000]
    al = CountingAllocator(A, torch)
    plain = al.alloc

    def _alloc(nbytes, stream, user):
        p = plain(nbytes, stream, user)
        if late and nbytes >= 340_000 * 256:
            with torch.cuda.stream(torch.cuda.ExternalStream(stream)):
                torch.cuda._sleep(20_000_000)
                al.live[p].fill_(0xA5)
        return p

    late = False
    al.inner, al.alloc = plain, A.ALLOC_FN(_alloc)
    first, second = torch.cuda.Stream(), torch.cuda.Stream()
    build = dict(seed=2, metric=A.MIPS, batch_cap=20_000, max_rounds=16)
    g, h = A.ann_build(old, 32, 32, 1.0, allocator=al, **build), A.ann_build(old, 32, 32, 1.0, **build)
    for pts in (old, x):
        if pts is x:
            A.ann_insert_points(g, x, 32, 1.0, seed=4)
            A.ann_insert_points(h, x, 32, 1.0, seed=4)
        want = A.ann_search(h, pts, q, 10, 32)
        torch.cuda.synchronize()
        late = True
        with torch.cuda.stream(first):
            torch.cuda._sleep(100_000_000)
            before = torch.cuda.Event()
            before.record()
            a = A.ann_search(g, pts, q, 10, 32)
            assert not before.query()
        with torch.cuda.stream(second):
            b = A.ann_search(g, pts, q, 10, 32)
        torch.cuda.synchronize()
        late = False
        for got in (a, b):
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


class _Limited:
    """An allocator that refuses one size or, from start() on, to hold more than `limit` bytes; counts the most it held
    from there on."""

    def __init__(self, A, limit=None, refuse=None):
        self.inner = A.TorchAllocator()
        self.size, self.held, self.most, self.limit, self.started = {}, 0, 0, limit, False

        def alloc(nbytes, stream, user):
            if nbytes == refuse or (self.started and limit is not None and self.held + nbytes > self.limit):
                return None
            p = self.inner.alloc(nbytes, stream, user)
            self.size[p] = nbytes
            self.held += nbytes
            self.most = max(self.most, self.held)
            return p

        def free(ptr, user):
            self.held -= self.size.pop(ptr)
            self.inner.free(ptr, user)

        self.alloc, self.free = A.ALLOC_FN(alloc), A.FREE_FN(free)

    def start(self, room=0):
        self.started, self.most = True, self.held
        if self.limit is not None:
            self.limit = max(self.limit, self.held + room)

    def fill(self, opts):
        opts.alloc = C.cast(self.alloc, C.c_void_p)
        opts.free = C.cast(self.free, C.c_void_p)
        opts.alloc_user = None


BUILD = dict(seed=2, batch_cap=20_000, max_rounds=16)


def _lost_lists(A, x, al):
    """visited lists that fit nowhere: their searches are repeated in memory that the build asks for then"""
    al.start()
    g = A.ann_build(x, 32, 64, 1.0, seed=2, metric=A.MIPS, allocator=al, batch_cap=60_000, visited_cap=16, spill_cap=1)
    return [g.neighbors()]


def _layered_queries(A, x, al):
    h = A.ann_hnsw_build(x, 16, 32, 1.0, metric=A.MIPS, allocator=al, **BUILD)
    al.start(room=x.shape[0] * 256)  # for the sketches or for what the call cannot do without
    return [t.cpu().numpy() for t in A.ann_hnsw_search(h, x, x[:20_000], 10, 32)]


def _insertion(A, x, al):
    old = x[:340_000]
    g = A.ann_build(old, 32, 32, 1.0, metric=A.MIPS, allocator=al, **BUILD)
    A.ann_search(g, old, x[:20_000], 10, 32)
    al.start()
    A.ann_insert_points(g, x, 32, 1.0, seed=4)
    return [g.neighbors()]


def _batch(A, x, al):
    g = A.ann_build(x, 32, 32, 1.0, metric=A.MIPS, allocator=al, **BUILD)
    A.ann_search(g, x, x[:20_000], 10, 32)
    ids = np.nonzero(g.neighbors()[:, 0] == 0xFFFFFFFF)[0].astype(np.uint32)
    al.start()
    A.ann_insert_batch(g, x, ids[ids != g.info().start][:40_000], 32, 1.0)
    return [g.neighbors()]


@pytest.mark.parametrize("calls,n", [(_lost_lists, 135_000), (_layered_queries, 345_000), (_insertion, 345_000), (_batch, 345_000)])
def test_what_fits_without_sketches_fits(env, calls, n):
    """Sketches take memory that nothing else wants: a call that succeeds where there is none for them succeeds
    where there is just as much in all."""
    torch, A, _ = env
    x = _points(torch, n, 200, "unit", 5)
    without = _Limited(A, refuse=(340_000 if calls is _insertion else n) * 256)
    want = calls(A, x, without)
    torch.cuda.synchronize()
    limited = _Limited(A, limit=without.most)
    got = calls(A, x, limited)
    for a, b in zip(want, got):
        assert np.array_equal(a, b)
    torch.cuda.synchronize()
    assert limited.held == 0


def test_few_searches_make_no_sketches(env):
    """Calls whose searches would not repay the sketches ask for no memory for them: few queries with wide beams, insertions
    into rows that the cache holds; with enough of them they do."""
    torch, A, _ = env
    n, d = (272 << 20) // 400, 100
    x = _points(torch, n, d, "unit", 9)
    refusing = _Refusing(A, n * 128)
    g = A.ann_build(x, 40, 32, 1.0, seed=2, allocator=refusing, batch_cap=20_000, max_rounds=16)
    assert refusing.refused == 1
    for nq, L, made in ((1500, 64, 0), (3000, 128, 0), (5000, 128, 0), (20_000, 10, 0), (20_000, 129, 0), (30_000, 64, 1)):
        before = refusing.refused
        A.ann_search(g, x, x[:nq], 10, L)
        assert refusing.refused - before == made, (nq, L)
    n = 300_010  # (no other array has the size of the sketches)
    for m, L in ((2500, 128), (6000, 64), (40_000, 64)):
        refusing = _Refusing(A, n * 128)
        g = A.ann_build(x[:n - m], 40, 16, 1.0, seed=2, allocator=refusing, batch_cap=20_000)
        A.ann_insert_points(g, x[:n], L, 1.0, seed=3)
        assert refusing.refused == 0, (m, L)
