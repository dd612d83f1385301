"""The one-workgroup sort of few keys, at the edges of its rows, instances and digit widths: stable on
the lowest bits of the key's upper word, like the sort by passes of several launches beyond it."""
import numpy as np
import pytest

from helpers import dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [1, 9, 10, 11, 18, 20, 32])
def test_few_keys(env, bits):
    torch, A, _ = env
    rng = np.random.default_rng(bits)
    for count in (2, 63, 64, 65, 1000, 1024, 1025, 4096, 4097, 8192, 8193, 12287, 12288, 12289):
        for distinct in (1, 7, 1 << min(bits, 31)):
            say(f"sort bits={bits} count={count} distinct={distinct}")
            dst = rng.integers(0, distinct, count).astype(np.uint64) & np.uint64((1 << bits) - 1)
            keys = (dst << np.uint64(32)) | np.arange(count, dtype=np.uint64)[::-1]
            keys[rng.random(count) < 0.1] = np.uint64(0xFFFFFFFFFFFFFFFF)  # empty places sort last
            t = dev(torch, keys.view(np.int64))
            A.ann_sort_edges(t, bits)
            want = keys[np.argsort((keys >> np.uint64(32)) & np.uint64((1 << bits) - 1), kind="stable")]
            assert (t.cpu().numpy().view(np.uint64) == want).all()
