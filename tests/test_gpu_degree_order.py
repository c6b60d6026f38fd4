"""The degree binning at the sizes where its blocks, wavefronts and prefix-sum chunks
end, checked by what a ranked handle gives back: a random labelling goes in by
vertex id, is stored by position in the degree order and must come back, into a
buffer filled with -1, for every vertex; and one step from it must equal the
oracle's, which needs hubs, lane rows and short rows in their classes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2411_19901_amd import lpa  # noqa: E402

pytestmark = pytest.mark.gpu


def skewed(n, seed):
    """Rows of 0 to 300 entries, most of them few; random, sorted columns."""
    rng = np.random.default_rng(seed)
    deg = np.minimum((rng.pareto(1.5, n) * 1.5).astype(np.int64), min(n, 300))
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(deg)
    key = np.repeat(np.arange(n, dtype=np.int64), deg) * n + rng.integers(0, n, rp[-1])
    key.sort()
    return rp, (key % n).astype(np.int32)


@pytest.mark.parametrize("n", [1, 64, 129, 513, 5000, 1 << 18, (1 << 18) + 1, 1 << 21,
                               (1 << 21) + 1])
def test_labels_come_back_and_step(n):
    rp, col = skewed(n, n)
    d = torch.device("cuda:0")
    s = lpa.LPA(torch.from_numpy(rp).to(d), torch.from_numpy(col).to(d), None, k=8, mode="det",
                lane_max_degree=64, ranked=True)
    rng = np.random.default_rng(n + 1)
    labels = rng.integers(0, n, n).astype(np.int32)
    flags = (rng.random(n) < 0.7).astype(np.uint8)
    s.set_state(labels, flags, 1)
    back = torch.full((n,), -1, dtype=torch.int32, device=d)
    act = torch.full((n,), 7, dtype=torch.uint8, device=d)
    assert lpa.lpa_get_state(s.h, back.data_ptr(), act.data_ptr(), False) == 1
    assert np.array_equal(back.cpu().numpy(), labels) and np.array_equal(act.cpu().numpy(), flags)
    changed, _ = s.step()
    want, _, dn, _ = oracle.lpa_move(rp, col, None, 8, False, labels, flags)
    back.fill_(-1)
    lpa.lpa_get_state(s.h, back.data_ptr(), act.data_ptr(), False)
    assert changed == dn and np.array_equal(back.cpu().numpy(), want)
    s.close()
