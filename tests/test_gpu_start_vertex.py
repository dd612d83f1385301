"""Start vertex of float rows: both kernels, at the edges of their workgroups (256 rows) and steps (16 columns)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d", [(1, 4), (255, 20), (256, 16), (257, 100), (2049, 36), (4100, 200), (600, 1024), (600, 1028), (700, 7)])
def test_float_start_vertex(env, n, d):
    torch, A, _ = env
    x = np.random.default_rng(n + d).standard_normal((n, d)).astype(np.float32)
    x[n // 2:] = x[:n - n // 2]  # every point twice: the smaller id wins
    # (the two best differ by far more than the 1e-16 of the fp64 sums; the mean's order of summation shifts them less still)
    s = ((x.astype(np.float64) - x.astype(np.float64).mean(0)) ** 2).sum(1)
    assert A.ann_start_vertex(torch.from_numpy(x).cuda()) == int(np.argmin(np.round(s, 9)))
