"""What the callbacks of the build options may rely on: when the library calls `free`, nothing that it queued
is still to run on that memory."""
import numpy as np
import pytest

from helpers import dev

pytestmark = pytest.mark.gpu


def _allocator(A, torch, stream):
    """Counts what is alive, runs dry `left` allocations from now, looks at the stream when memory comes back."""
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
