"""The largest number of vertices that lpa_init takes, 2^31 - 2, nearly all of them
isolated: kernels that walk the vertices step past the range of int there."""
import pytest

torch = pytest.importorskip("torch")

from paper_2411_19901_amd import lpa  # noqa: E402

pytestmark = pytest.mark.gpu


def is_iota(x, step=1 << 28):
    return all(torch.equal(x[b:b + step],
                           torch.arange(b, min(b + step, x.numel()), dtype=torch.int32,
                                        device=x.device))
               for b in range(0, x.numel(), step))


@pytest.mark.timeout(120)
@pytest.mark.parametrize("ranked", [False, True])
def test_two_last_vertices_of_the_most(ranked):
    n = 2 ** 31 - 2
    dev = torch.device("cuda:0")
    rp = torch.zeros(n + 1, dtype=torch.int32, device=dev)  # one edge, n - 2 to n - 1
    rp[n - 1] = 1
    rp[n] = 2
    col = torch.tensor([n - 1, n - 2], dtype=torch.int32, device=dev)
    s = lpa.LPA(rp, col, None, k=8, mode="det", max_iter=4, ranked=ranked)
    assert is_iota(s.labels())
    s.step()  # pick-less: only n - 1 may move, to the lower label
    got = s.labels()
    assert int(got[n - 1]) == n - 2 and is_iota(got[:n - 1])
    # the pair is one community with all of the weight: Q = 1 - 1
    assert s.modularity() == 0.0 and s.modularity(got) == 0.0
    s.close()
    del rp, col, got, s
    torch.cuda.empty_cache()
