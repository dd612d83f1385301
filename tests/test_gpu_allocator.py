"""What the callbacks of the build options may rely on: when the library calls `free`, nothing that it queued
is still to run on that memory, also where the call fails half-way; `alloc` is asked for memory on the stream of
the call that needs it, and what it gives is first used there."""
import numpy as np
import pytest

from helpers import dev, say

pytestmark = pytest.mark.gpu


def _allocator(A, torch, stream):
    """Counts what is alive, runs dry where a test says so, looks at the stream when memory comes back."""
    from test_gpu_boundary import CountingAllocator

    class Watching(CountingAllocator):
        def __init__(self):
            super().__init__(A, torch)
            self.busy = 0
            give_back = self.free

            def _free(ptr, user):
                self.busy += 0 if stream.query() else 1
                give_back(ptr, user)

            self.inner, self.free = give_back, A.FREE_FN(_free)

    return Watching()


def _calls(A, pts):
    """call -> (what is there before it, the call)"""
    half = pts[:pts.shape[0] // 2]
    return {
        "build": (lambda al: None, lambda g, al: A.ann_build(pts, 16, 32, 1.2, seed=3, allocator=al)),
        "insert": (lambda al: A.ann_build(half, 16, 32, 1.2, seed=3, allocator=al),
                   lambda g, al: A.ann_insert_points(g, pts, 32, 1.2, seed=4)),
        "layered": (lambda al: None, lambda g, al: A.ann_hnsw_build(pts, 8, 32, 1.2, seed=3, allocator=al)),
        "layered insert": (lambda al: A.ann_hnsw_build(half, 8, 32, 1.2, seed=3, allocator=al),
                           lambda g, al: A.ann_hnsw_insert_points(g, pts, 32, 1.2, seed=4)),
        "cluster": (lambda al: None, lambda g, al: A.ann_hcnng_build(pts, 3, 100, 3, 10, 16, 1.2, seed=3, allocator=al)),
    }


@pytest.mark.parametrize("call", ["build", "insert", "layered", "layered insert", "cluster"])
def test_memory_comes_back_idle(env, call):
    """Padded byte rows (a copy of the points is one more allocation).  Work queued before the call keeps
    everything that the call queues from running until somebody waits."""
    torch, A, _ = env
    pts = dev(torch, np.random.default_rng(5).integers(0, 256, (1500, 60)).astype(np.uint8))
    before, act = _calls(A, pts)[call]
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        def once(k):
            """with k allocations (None: all that it wants); returns how many the call made"""
            al = _allocator(A, torch, stream)
            g = before(al)
            stream.synchronize()
            had = al.allocs
            if k is None:
                made = act(g, al)
            else:
                al.fail_after = had + k
                torch.cuda._sleep(5_000_000)  # some milliseconds
                with pytest.raises(A.AnnError) as e:
                    act(g, al)
                assert e.value.code == -2
                made = e = None
            assert al.busy == 0, f"{al.busy} buffers came back with work queued"
            n = al.allocs - had
            stream.synchronize()  # (an object that is freed does not wait for the caller's searches)
            del made, g
            assert len(al.live) == 0 and al.allocs == al.frees
            return n

        total = once(None)
        for k in range(total):
            say(f"allocator {call}: dry after {k} of {total}")
            assert once(k) == k


def test_layered_insert_waits_for_searches(env):
    """An insertion that nothing has to grow for replaces the table that a search in flight reads."""
    torch, A, _ = env
    pts = dev(torch, np.random.default_rng(6).integers(0, 256, (1000, 64)).astype(np.uint8))
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        al = _allocator(A, torch, stream)
        h = A.ann_hnsw_build(pts[:600], 8, 32, 1.2, seed=3, allocator=al)
        assert h.info().top > 0
        A.ann_hnsw_insert_points(h, pts[:610], 32, 1.2, seed=4)  # (room for 900 points from here on)
        want, _ = A.ann_hnsw_search(h, pts[:610], pts[:50], 5, 20)
        stream.synchronize()
        al.busy = 0
        torch.cuda._sleep(5_000_000)
        ids, _ = A.ann_hnsw_search(h, pts[:610], pts[:50], 5, 20)
        A.ann_hnsw_insert_points(h, pts[:700], 32, 1.2, seed=5, level=np.zeros(90, np.uint32))
        assert al.busy == 0 and torch.equal(ids, want)
        stream.synchronize()
        del h


def test_layered_queries_after_one_that_failed(env):
    """A call that finds no room for its start vertices has given up the smaller array of the calls before."""
    torch, A, _ = env
    pts = dev(torch, np.random.default_rng(10).integers(0, 256, (1000, 64)).astype(np.uint8))
    al = _allocator(A, torch, torch.cuda.current_stream())
    h = A.ann_hnsw_build(pts, 8, 32, 1.2, seed=3, allocator=al)
    assert h.info().top > 0
    want, _ = A.ann_hnsw_search(h, pts, pts[:50], 5, 20)
    al.fail_after = al.allocs
    with pytest.raises(A.AnnError) as e:
        A.ann_hnsw_search(h, pts, pts[:500], 5, 20)
    assert e.value.code == -2
    al.fail_after = None
    ids, _ = A.ann_hnsw_search(h, pts, pts[:50], 5, 20)
    assert torch.equal(ids, want)


def test_layered_index_after_an_insertion_that_failed(env):
    """Wherever an insertion runs dry, the index answers as before, answers over the points that it holds, or refuses."""
    torch, A, _ = env
    pts = dev(torch, np.random.default_rng(11).integers(0, 256, (1500, 60)).astype(np.uint8))
    stream = torch.cuda.current_stream()

    def once(k):
        al = _allocator(A, torch, stream)
        h = A.ann_hnsw_build(pts[:600], 8, 32, 1.2, seed=3, allocator=al)
        assert h.info().top > 0
        want, _ = A.ann_hnsw_search(h, pts, pts[:50], 5, 20)
        had = al.allocs
        al.fail_after = None if k is None else had + k
        try:
            A.ann_hnsw_insert_points(h, pts, 32, 1.2, seed=4)
            assert k is None
            return al.allocs - had
        except A.AnnError as e:
            assert e.code == -2
        al.fail_after = None
        try:
            ids, _ = A.ann_hnsw_search(h, pts, pts[:50], 5, 20)
            h.layer(1)
        except A.AnnError as e:
            assert e.code == -1 and k > 1 and "can only be freed" in str(e)
            for again in (lambda: h.layer(1), lambda: A.ann_hnsw_insert_points(h, pts, 32, 1.2, seed=4)):
                with pytest.raises(A.AnnError):
                    again()
            return "refused"
        if h.info().n == 600:
            assert k < 2 and torch.equal(ids, want)  # (the bottom layer's rows and degrees)
        else:
            assert h.info().n == 1500 and (ids >= 0).all() and (ids < 1500).all()
        return "answered"

    total = once(None)
    seen = set()
    for k in range(total):
        say(f"layered insertion dry after {k} of {total}")
        seen.add(once(k))
    assert seen == {"refused", "answered"}


def test_alloc_names_the_stream_of_the_call(env):
    """Searches and insertions on another stream than the build's: padded copies, grown rows, scratch, start vertices."""
    from test_gpu_boundary import CountingAllocator
    torch, A, _ = env
    pts = dev(torch, np.random.default_rng(7).integers(0, 256, (1200, 60)).astype(np.uint8))
    al = CountingAllocator(A, torch)
    plain, asked = al.alloc, []

    def _alloc(nbytes, stream, user):
        asked.append(stream or 0)
        return plain(nbytes, stream, user)

    al.inner, al.alloc = plain, A.ALLOC_FN(_alloc)
    first, second = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(first):
        g = A.ann_build(pts[:600], 16, 32, 1.2, seed=3, allocator=al)
        h = A.ann_hnsw_build(pts[:600], 8, 32, 1.2, seed=3, allocator=al)
    assert set(asked) == {first.cuda_stream}
    calls = {
        "search": lambda: A.ann_search(g, pts[:600], pts[:100], 5, 20),
        "reserve": lambda: A.ann_graph_reserve(g, 700),
        "insert": lambda: A.ann_insert_points(g, pts, 32, 1.2, seed=4),
        "layered search": lambda: A.ann_hnsw_search(h, pts[:600], pts[:100], 5, 20),
        "layered insert": lambda: A.ann_hnsw_insert_points(h, pts, 32, 1.2, seed=4),
    }
    for name, call in calls.items():
        del asked[:]
        with torch.cuda.stream(second):
            call()
        assert asked and set(asked) == {second.cuda_stream}, name
    torch.cuda.synchronize()
    del g, h, calls, call
    assert len(al.live) == 0


def test_memory_is_first_used_on_its_stream(env):
    """Memory that comes with work of its last owner still queued on the stream: fills that run late.
    Rows that are padded, a batch whose visited lists fit nowhere (more allocations), every builder."""
    from test_gpu_boundary import CountingAllocator
    torch, A, _ = env
    pts = dev(torch, np.random.default_rng(8).integers(0, 256, (1500, 60)).astype(np.uint8))
    half = pts[:700]
    al = CountingAllocator(A, torch)
    plain = al.alloc

    def _alloc(nbytes, stream, user):
        p = plain(nbytes, stream, user)
        with torch.cuda.stream(torch.cuda.ExternalStream(stream)):
            torch.cuda._sleep(300_000)
            al.live[p].fill_(0xA5)
        return p

    al.inner, al.alloc = plain, A.ALLOC_FN(_alloc)

    def everything(a):
        out = []
        g = A.ann_build(half, 16, 40, 1.2, seed=3, allocator=a, visited_cap=16, spill_cap=1)
        out.append(g.neighbors())
        A.ann_insert_points(g, pts, 40, 1.2, seed=4)
        out += [g.neighbors(), *A.ann_search(g, pts, pts[:300], 5, 20)]
        first = A.ann_build(half, 16, 40, 1.2, seed=3, allocator=a, max_rounds=4)
        ids = np.nonzero(first.neighbors()[:, 0] == 0xFFFFFFFF)[0].astype(np.uint32)
        A.ann_insert_batch(first, half, ids[ids != first.info().start][:50], 40, 1.2)
        out.append(first.neighbors())
        h = A.ann_hnsw_build(half, 8, 40, 1.2, seed=3, allocator=a)
        A.ann_hnsw_insert_points(h, pts, 40, 1.2, seed=4)
        out += [l for i in range(h.info().top + 1) for l in h.layer(i)]
        out += A.ann_hnsw_search(h, pts, pts[:300], 5, 20)
        out.append(A.ann_hcnng_build(pts, 3, 100, 3, 10, 16, 1.2, seed=3, allocator=a).neighbors())
        torch.cuda.synchronize()
        return out

    want = everything("torch")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        got = everything(al)
    for w, x in zip(want, got):
        assert torch.equal(w, x) if isinstance(w, torch.Tensor) else (w == x).all()
    assert len(al.live) == 0


@pytest.mark.parametrize("dtype,d,n,T,Ls,l", [("uint8", 128, 40000, 6, 1000, 10), ("int8", 40, 20000, 5, 100, 16), ("float32", 256, 20000, 4, 500, 16),
                                             ("uint8", 128, 20000, 3, 8, 4)])
def test_cluster_build_holds_what_the_header_says(env, dtype, d, n, T, Ls, l):
    """ann_hcnng_opts names the bytes that a build holds while it runs."""
    from test_gpu_boundary import CountingAllocator
    torch, A, _ = env
    rng = np.random.default_rng(9)
    pts = dev(torch, rng.standard_normal((n, d)).astype(dtype) if dtype == "float32" else rng.integers(0, 100, (n, d)).astype(dtype))
    al = CountingAllocator(A, torch)
    plain, live, held = al.alloc, {}, [0]
    give_back = al.free

    def _alloc(nbytes, stream, user):
        p = plain(nbytes, stream, user)
        live[p] = nbytes
        held[0] = max(held[0], sum(live.values()))
        return p

    def _free(ptr, user):
        del live[ptr]
        give_back(ptr, user)

    al.inner, al.alloc, al.free = (plain, give_back), A.ALLOC_FN(_alloc), A.FREE_FN(_free)
    R = 24
    g = A.ann_hcnng_build(pts, T, Ls, 3, l, R, 1.2, seed=3, allocator=al)
    row = d * pts.element_size()
    stride, G = (row + 31) // 32 * 32, max(1, min(T, (1 << 25) // n))
    said = (28 + 6 * l + stride * (1 + 128 / Ls) + 100 / Ls) * G * n + 33 * T * n + 48 * n
    graph = n * (4 * R + 4) + (1 << 21)
    padded = n * 2 * row if dtype != "float32" and d % 16 else 0
    assert 0.9 * said < held[0] < 1.01 * said + graph + padded, (held[0], said)
    del g
