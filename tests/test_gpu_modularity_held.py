"""Modularity of labellings in which a label takes over in the middle of the degree
order, so that wavefronts hold one label's sum, give it up for another's and add
the rest lane by lane, against the oracle in fp64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2411_19901_amd import inputs  # noqa: E402
from test_gpu_batch import dev, make_solver  # noqa: E402

pytestmark = pytest.mark.gpu


def labelling(kind, n, rng):
    v = np.arange(n)
    r = rng.random(n)
    if kind == "half in one":
        return np.where(r < 0.5, n - 1, np.where(r < 0.8, v // 16 * 16, v))
    if kind == "two in turn":  # a quarter each, the more frequent one by id range
        return np.where(r < 0.2 + 0.3 * ((v // 97) % 2), 0, np.where(r < 0.6, n // 2, v))
    if kind == "seven of 64":  # just short of the eight that a label needs
        return np.where(v % 64 < 7, 1, v)
    return np.where(v % 64 < 8, 1, v)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("kind", ["half in one", "two in turn", "seven of 64", "eight of 64"])
@pytest.mark.parametrize("name", ["rmat", "sbm", "grid"])
def test_against_oracle(name, kind, weighted):
    g = {"rmat": lambda: inputs.rmat(13), "sbm": lambda: inputs.sbm1(3),
         "grid": lambda: inputs.grid(90, 71, 0.05, 0.01, seed=2)}[name]()
    if weighted:
        g = inputs.with_uniform_weights(g, 4)
    lab = labelling(kind, g.n, np.random.default_rng(5)).astype(np.int32)
    s = make_solver(g)
    got = s.modularity(torch.from_numpy(lab).to(dev()))
    # Q = sigma / 2m - sum(tot^2) / (2m)^2, both terms at most 1; each of the sums has at
    # most nnz non-negative fp64 terms, so nnz * 2^-53 relative: 2 of them in the first
    # term, 4 in the second, on either side
    assert abs(got - oracle.modularity(g.row_ptr, g.col, g.w, lab)) <= 12 * g.nnz * 2.0 ** -53
    s.close()
