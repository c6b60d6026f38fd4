"""The det mode's default lane threshold depends on the graph's entry count.
Graphs with one edge less than, and exactly, each count at which it changes,
with rows on both sides of both thresholds, give the oracle's labels and
counts bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2411_19901_amd import inputs  # noqa: E402
from test_gpu_parity import check_det  # noqa: E402

pytestmark = pytest.mark.gpu

N = 40_000


def skewed(m, seed=11):
    """m distinct edges, one end drawn towards the low ids."""
    rng = np.random.default_rng(seed)
    u = (N * rng.random(2 * m + 4096) ** 4).astype(np.int64)
    v = rng.integers(0, N, u.size)
    keys = np.unique(np.minimum(u, v)[u != v] * N + np.maximum(u, v)[u != v])
    keys = np.sort(rng.permutation(keys)[:m])
    assert keys.size == m
    return inputs.with_uniform_weights(
        inputs.from_edges(N, np.stack([keys // N, keys % N], 1), name=f"skewed{m}"), seed)


@pytest.mark.parametrize("below", [1, 0])
@pytest.mark.parametrize("log2_nnz,small,large", [(18, 64, 128), (20, 128, 256), (21, 256, 768)])
def test_det_parity_at_default_threshold(log2_nnz, small, large, below):
    g = skewed((1 << (log2_nnz - 1)) - below)
    d = np.diff(g.row_ptr)
    assert g.nnz == (1 << log2_nnz) - 2 * below
    assert (d > large).any() and ((d > small) & (d <= large)).any() and (d <= small).any()
    check_det(g, 8)
