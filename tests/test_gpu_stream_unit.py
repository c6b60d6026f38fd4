"""Streamed unit-weight graphs of many ranges with few unprocessed vertices: most
lanes of a wavefront have no entries of their own, and the ranges lie far past
the four slice buffers.  Each step must equal the oracle's from the same state."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2411_19901_amd import lpa  # noqa: E402
from test_gpu_parity import graph  # noqa: E402
from test_gpu_stream import pinned  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offsets64", [False, True])
@pytest.mark.parametrize("variant", [dict(k=1), dict(k=8), dict(k=8, lane_max_degree=16),
                                     dict(k=1, rule="bm_paper")])
@pytest.mark.parametrize("share", [0.02, 0.5])
def test_sparse_steps_match_oracle(share, variant, offsets64):
    g = graph("sbm1-iso")
    rp, col, _ = pinned(g, offsets64)
    s = lpa.LPA(rp, col, None, mode="det", stream_csr=True, stream_chunk_kib=1, **variant)
    rule = oracle.BM_PAPER if "rule" in variant else variant["k"]
    rng = np.random.default_rng(int(100 * share))
    labels = np.arange(g.n, dtype=np.int32)
    for it in (1, 2, 8):
        flags = (rng.random(g.n) < share).astype(np.uint8)
        s.set_state(labels, flags, it)
        changed, _ = s.step()
        want, _, dn, _ = oracle.lpa_move(g.row_ptr, g.col, None, rule, it % 8 == 0, labels, flags)
        labels = s.get_state()[0]
        assert changed == dn and np.array_equal(labels, want), it
    s.close()


@pytest.mark.parametrize("offsets64", [False, True])
def test_async_scans_every_entry(offsets64):
    g = graph("sbm1-iso")
    rp, col, _ = pinned(g, offsets64)
    s = lpa.LPA(rp, col, None, k=8, mode="async", stream_csr=True, stream_chunk_kib=1,
                lane_max_degree=16)
    s.run()
    lab = s.labels(device=False)
    assert lab.min() >= 0 and lab.max() < g.n
    assert s.trace()[1][0] == g.nnz
    s.close()
