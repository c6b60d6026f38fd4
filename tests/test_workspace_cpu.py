"""lpa_workspace_bytes never decreases as a graph grows, so that one workspace
sized for a caller's largest graph holds every smaller one (no GPU needed)."""
import pytest

from paper_2411_19901_amd import lpa


@pytest.mark.parametrize("kw", [dict(mode="det"), dict(mode="det", rescan=True),
                                dict(mode="det", ranked=True), dict(mode="det", k=32),
                                dict(mode="det", lane_max_degree=64), dict(mode="async")])
@pytest.mark.parametrize("n", [5_000, 40_000, 3_000_000])
def test_bytes_do_not_decrease_with_entries(n, kw):
    counts = sorted({c for e in (10, 18, 20, 21, 24, 28)
                     for c in ((1 << e) - 1, 1 << e, (1 << e) + 1, 3 << (e - 1))})
    sizes = [lpa.workspace_bytes(n, c, **kw) for c in counts]
    assert sizes == sorted(sizes), list(zip(counts, sizes))


@pytest.mark.parametrize("nnz", [0, 1000, 1 << 22])
def test_bytes_do_not_decrease_with_vertices(nnz):
    counts = sorted({c for e in (0, 9, 10, 18, 21, 22, 23)
                     for c in ((1 << e) - 1, 1 << e, (1 << e) + 1)} - {0})
    sizes = [lpa.workspace_bytes(c, nnz) for c in counts]
    assert sizes == sorted(sizes), list(zip(counts, sizes))
