"""The one-wavefront-per-hub chains of det mode at the lengths where they can
go wrong: rows around the queue's 64-entry blocks and the 256-entry chunks,
with labels that all differ, that share one heavy label (whose entries the
unit-weight chain counts apart), two heavy labels in turn, or few labels (most
entries are hits), repeated neighbours and entries of the vertex itself.  One
step from a restored state must give the oracle's labels bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2411_19901_amd import lpa  # noqa: E402

pytestmark = pytest.mark.gpu

LENGTHS = [2, 7, 8, 9, 63, 64, 65, 127, 255, 256, 257, 319, 320, 321, 385, 1000, 4099]
LEAVES = 5000


def hub_graph(distinct, seed):
    """Hubs 0 .. 4 H - 1 (every length with four kinds of labels) over LEAVES
    vertices that have no row of their own; labels of the leaves by kind."""
    rng = np.random.default_rng(seed)
    hubs = [(n, kind) for n in LENGTHS for kind in range(4)]
    H = len(hubs)
    n = H + 4 * LEAVES
    lab = np.arange(n)
    r = rng.random(LEAVES)
    some = H + LEAVES * np.arange(4)
    lab[some[1]:some[2]] = np.where(r < 0.4, 17, lab[some[1]:some[2]])
    turn = np.arange(LEAVES) % 1500 < 750
    lab[some[2]:some[3]] = np.where(r < 0.7, np.where(turn, 5, 9), lab[some[2]:some[3]])
    lab[some[3]:] = rng.integers(0, 12, LEAVES)
    rows = []
    for v, (m, kind) in enumerate(hubs):
        ids = some[kind] + np.arange(LEAVES)
        row = np.sort(rng.choice(ids, m, replace=not distinct))
        if m % 2:  # the vertex itself, in order
            row[0] = v
        rows.append(row)
    rp = np.zeros(n + 1, np.int32)
    rp[1:H + 1] = np.cumsum([len(x) for x in rows])
    rp[H + 1:] = rp[H]
    w = (rng.integers(1, 1 << 24, rp[-1]) * 2.0 ** -24).astype(np.float32)
    return rp, np.concatenate(rows).astype(np.int32), w, lab.astype(np.int32), n


@pytest.mark.parametrize("ranked", [False, True])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("k", [1, 2, 4, 8, 16, 32])
def test_hub_chains_match_the_oracle(k, weighted, ranked):
    rp, col, w, lab, n = hub_graph(False, 10 + k)
    w = w if weighted else None
    dev = torch.device("cuda:0")
    s = lpa.LPA(torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev),
                None if w is None else torch.from_numpy(w).to(dev), k=k, mode="det", tol=0.0,
                max_iter=4, lane_max_degree=1, ranked=ranked)
    act = np.ones(n, np.uint8)
    s.set_state(lab, act, 1)
    changed, _ = s.step()
    want, _, dn, _ = oracle.lpa_move(rp, col, w, k, False, lab, act)
    assert np.array_equal(s.labels(device=False), want)
    assert changed == dn
    s.close()


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("k", [1, 4, 8, 32])
def test_first_iteration_of_rows_without_repeats(k, weighted):
    rp, col, w, _, n = hub_graph(True, 50 + k)
    w = w if weighted else None
    dev = torch.device("cuda:0")
    s = lpa.LPA(torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev),
                None if w is None else torch.from_numpy(w).to(dev), k=k, mode="det", tol=0.0,
                max_iter=4, lane_max_degree=1, rho=0)
    s.step()
    lab = np.arange(n, dtype=np.int32)
    want, _, _, _ = oracle.lpa_move(rp, col, w, k, False, lab, np.ones(n, np.uint8))
    assert np.array_equal(s.labels(device=False), want)
    s.close()
