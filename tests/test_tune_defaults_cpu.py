"""The autotuner times every threshold that the library takes by default, so a graph
for which the default is the fastest keeps it."""
import numpy as np
import pytest

from paper_2411_19901_amd import inputs, tune

# lane_max_degree = 0 in include/lpa.h: async, and det by the number of entries
DEFAULTS = {"async": (1024,), "det": (64, 128, 256, 768, 2048)}


@pytest.mark.parametrize("mode,best", [(m, s) for m, v in DEFAULTS.items() for s in v])
def test_default_threshold_is_a_candidate(monkeypatch, mode, best):
    g = inputs.rmat(12)  # its largest row is longer than half of every default
    assert 2 * int(np.diff(g.row_ptr).max()) >= max(max(v) for v in DEFAULTS.values())
    monkeypatch.setattr(tune, "arch_name", lambda device=None: "")
    monkeypatch.setattr(tune, "_time_config",
                        lambda lpa, torch, rp, col, w, cfg, *rest:
                        1.0 if cfg["lane_max_degree"] == best else 2.0)
    r = tune.tune(g.row_ptr, g.col, None, mode=mode)
    assert r["lane_max_degree"] == best
