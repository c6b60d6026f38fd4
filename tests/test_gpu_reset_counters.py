"""lpa_reset clears the counters of every iteration, however many a handle may run:
a second solve counts the same changed vertices and scanned entries as the first."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2411_19901_amd import inputs, lpa  # noqa: E402
from test_gpu_batch import dev, make_solver  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("max_iter", [1, 255, 256, 257, 3000])
def test_counts_of_a_second_solve(max_iter, batched):
    g = inputs.sbm1(1)  # tol 0: runs all its iterations
    stream = torch.cuda.current_stream(dev())
    s = make_solver(g, tol=0.0, max_iter=max_iter, stream=stream)
    batch = lpa.Batch(1, k=8, mode="det", stream=stream)
    s.run()
    dn, sc = s.trace()
    if batched:
        batch.reset([s])
        batch.run([s])
    else:
        s.reset()
        s.run()
    dn2, sc2 = s.trace()
    assert len(dn) == len(dn2) and np.array_equal(dn, dn2) and np.array_equal(sc, sc2)
    batch.close()
    s.close()
