"""Stage times of a setup: every stage has its own, and they make up the total."""

import pytest

from gpu_helpers import setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("params", [{}, {"sweeps": 1}, {"sweeps": 8}, {"smooth_p": 1}])
@pytest.mark.parametrize("name", ["grid", "graph"])
def test_stages(name, params):
    from paper_2006_16147_amd import inputs

    # (the graph stops coarsening in the middle of a level's sweeps)
    A = inputs.laplacian7(64) if name == "grid" else inputs.random_spd_graph(
        3000, 3.0 if "smooth_p" in params else 6.0, seed=2)
    setup(A, **params).close()  # the library's first memory of this size
    h = setup(A, **params)
    t = h.setup_times()
    stages = {k: v for k, v in t.items() if k != "total"}
    assert min(stages.values()) > 0.0, t
    assert 0.8 * t["total"] <= sum(stages.values()) <= 1.001 * t["total"], t
    h.close()
