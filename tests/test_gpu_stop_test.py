"""Solves on both sides of the sizes up to which the move kernel runs the stop test
itself (128 workgroups of four items, 256 graphs): iterations, changed and
scanned counts and labels must equal the oracle's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2411_19901_amd import inputs, lpa  # noqa: E402
from test_gpu_batch import dev, make_solver  # noqa: E402

pytestmark = pytest.mark.gpu


def check(g, s):
    ref, rit, rdn, rsc = oracle.lpa_run(g.row_ptr, g.col, g.w, k=8)
    dn, sc = s.trace()
    assert s.iterations() == rit and np.array_equal(dn, rdn) and np.array_equal(sc, rsc)
    assert np.array_equal(s.labels(device=False), ref)


@pytest.mark.parametrize("items", [508, 512, 513, 520, 1024])
@pytest.mark.parametrize("check_every", [0, 3])
def test_workgroups(items, check_every):
    n, m = 64 * items, 3  # rows of six entries: 64 to an item, no short ones
    rng = np.random.default_rng(items)
    off = np.concatenate([np.arange(-m, 0), np.arange(1, m + 1)])
    col = np.sort((np.arange(n)[:, None] + off) % n, axis=1).astype(np.int32).reshape(-1)
    g = inputs.Graph(np.arange(n + 1, dtype=np.int32) * 2 * m, col,
                     rng.random(n * 2 * m, dtype=np.float32) + np.float32(0.5), "ring")
    s = make_solver(g, check_every=check_every)
    for _ in range(2):
        s.reset()
        s.run()
        check(g, s)
    s.reset()
    while not s.step()[1]:
        pass
    check(g, s)
    s.close()


@pytest.mark.parametrize("count", [255, 256, 257, 600])
def test_graphs(count):
    stream = torch.cuda.current_stream(dev())
    pool = [inputs.batch_graph(s, 9, i) for i, s in enumerate(inputs.batch_specs(8, 9, 60, 100))]
    solvers = [make_solver(pool[i % 8], stream=stream) for i in range(count)]
    batch = lpa.Batch(count, k=8, mode="det", stream=stream)
    for _ in range(2):
        batch.reset(solvers)
        batch.run(solvers)
    for i, s in enumerate(solvers):
        check(pool[i % 8], s)
        s.close()
    batch.close()
