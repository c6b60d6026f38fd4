"""Batched resets of different sets of graphs one after another, all queued behind
earlier work of the stream: each reset must reach the graphs it was called for,
whatever the calls after it upload."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2411_19901_amd import lpa  # noqa: E402
from test_gpu_batch import dev, make_solver, mixed_graphs, oracle_labels  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("capacity", [12, 2000])  # tables uploaded in one copy, in two
@pytest.mark.parametrize("resets", [1, 2, 3])
def test_resets_behind_queued_work(resets, capacity):
    gs = mixed_graphs(count=9, seed=23)
    sets = [gs[:6], gs[6:8], gs[8:]]
    stream = torch.cuda.current_stream(dev())
    solvers = [[make_solver(g, stream=stream) for g in part] for part in sets]
    batch = lpa.Batch(capacity, k=8, mode="det", stream=stream)
    for part in solvers:
        batch.run(part)
    torch.cuda._sleep(50_000_000)  # some 20 ms: the uploads below wait behind it
    for part in solvers[:resets]:
        batch.reset(part)
    for part, graphs in zip(solvers[:resets], sets):
        for s in part:
            assert s.iterations() == 0
        batch.run(part)
        for s, g in zip(part, graphs):
            ref, rit, rdn, rsc = oracle_labels(g)
            assert s.iterations() == rit, g.name
            dn, sc = s.trace()
            assert np.array_equal(dn, rdn) and np.array_equal(sc, rsc), g.name
            assert np.array_equal(s.labels(device=False), ref), g.name
    batch.close()
    for part in solvers:
        for s in part:
            s.close()
