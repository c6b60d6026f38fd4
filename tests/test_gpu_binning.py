"""The degree binning at the sizes where its blocks, wavefronts and prefix-sum
chunks end: the degree order must list every vertex once.  With the ranked
layout each vertex's state lies at its position in that order, so right after
lpa_init the labels come back as the vertex ids only if it does."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2411_19901_amd import lpa  # noqa: E402

pytestmark = pytest.mark.gpu


def skewed(n, seed):
    """Rows of skewed lengths (0 to about 1000) with random, sorted columns."""
    rng = np.random.default_rng(seed)
    deg = np.minimum((rng.pareto(1.1, n) * 2).astype(np.int64), min(n, 1000))
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(deg)
    col = rng.integers(0, n, rp[-1]).astype(np.int32)
    row = np.repeat(np.arange(n), deg)
    return rp, col[np.lexsort((col, row))]


@pytest.mark.parametrize("n", [1, 63, 64, 127, 128, 129, 511, 512, 513, 5000, 1 << 18,
                               (1 << 18) + 1, (1 << 21) - 1, (1 << 21) + 1])
def test_degree_order_lists_every_vertex_once(n):
    rp, col = skewed(n, n)
    dev = torch.device("cuda:0")
    s = lpa.LPA(torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), None, mode="det",
                lane_max_degree=64, ranked=True, max_iter=1)
    assert np.array_equal(s.labels(device=False), np.arange(n))
    if n < 1 << 17:  # hubs, lane rows and short rows each get the rows that are theirs
        s.step()
        want = oracle.lpa_run(rp, col, None, k=8, max_iter=1)[0]
        assert np.array_equal(s.labels(device=False), want)
    s.close()
