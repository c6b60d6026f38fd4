"""Det solves of small graphs in one launch, one workgroup of 16 wavefronts per
graph: at most 17 work items of 64 (or, for the rows of at most 4 entries, 128)
vertices.  Graphs on both sides of that limit, alone, in a batch, captured, in
single steps and resumed from a saved state give the oracle's labels, iteration
count and per-iteration counts bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2411_19901_amd import inputs, lpa  # noqa: E402
from test_gpu_parity import check_det, to_dev  # noqa: E402

pytestmark = pytest.mark.gpu


def sbm(n, weights, seed=3):
    rng = np.random.default_rng(seed + n)
    m = 7 * n
    u = rng.integers(0, n, m)
    v = np.where(rng.random(m) < 0.85, (u // 50) * 50 + rng.integers(0, 50, m),
                 rng.integers(0, n, m)).clip(0, n - 1)
    keys = np.unique(np.minimum(u, v)[u != v] * n + np.maximum(u, v)[u != v])
    g = inputs.from_edges(n, np.stack([keys // n, keys % n], 1), name=f"s{n}")
    return inputs.with_uniform_weights(g, seed) if weights else g


@pytest.mark.parametrize("n", [2, 63, 64, 65, 1000, 1023, 1024, 1025, 1100, 1300])
@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("k", [1, 2, 4, 8, 16])
def test_det_parity(n, weights, k):
    check_det(sbm(n, weights), k)


def solve(s):
    it = s.run()
    return it, s.labels(device=False), [x.tolist() for x in s.trace()]


def check(s, g, **kw):
    it, lab, (dn, sc) = solve(s)
    ref, rit, rdn, rsc = oracle.lpa_run(g.row_ptr, g.col, g.w, k=8, **kw)
    assert it == rit and dn == list(rdn) and sc == list(rsc)
    assert np.array_equal(lab, ref)


@pytest.mark.parametrize("kw", [dict(rho=0), dict(tol=0.0), dict(max_iter=2), dict(max_iter=1)])
@pytest.mark.parametrize("option", [dict(), dict(ranked=True), dict(check_every=1),
                                    dict(capture=True)])
def test_det_parity_options(kw, option):
    g = sbm(777, True)
    rp, col, w = to_dev(g)
    s = lpa.LPA(rp, col, w, k=8, **kw, **option)
    for _ in range(3):  # a captured run is replayed
        check(s, g, **kw)
        s.reset()
    s.close()


@pytest.mark.parametrize("capture", [False, True])
@pytest.mark.parametrize("n", [(900, 70, 500, 1024), (900, 70, 500, 2000)])
def test_batches_with_a_finished_graph(capture, n):
    gs = [sbm(x, False) for x in n]
    solvers = [lpa.LPA(*to_dev(g), k=8) for g in gs]
    b = lpa.Batch(len(gs), k=8, capture=capture)
    solvers[1].run()  # finished before the batch runs
    for _ in range(3):
        b.run(solvers)
        for s, g in zip(solvers, gs):
            assert s.finished()
            check(s, g)  # a finished graph's run changes nothing
        b.reset(solvers)


def test_steps_and_saved_state():
    g = sbm(1000, True)
    rp, col, w = to_dev(g)
    whole = lpa.LPA(rp, col, w, k=8)
    it, lab, (dn, sc) = solve(whole)
    a = lpa.LPA(rp, col, w, k=8)
    b = lpa.LPA(rp, col, w, k=8)
    assert [a.step()[0] for _ in range(2)] == dn[:2]
    b.set_state(*a.get_state())
    for s, skip in ((a, 0), (b, 2)):
        i, l, t = solve(s)
        assert i == it and np.array_equal(l, lab)
        assert t[0][skip:] == dn[skip:] and t[1][skip:] == sc[skip:]
