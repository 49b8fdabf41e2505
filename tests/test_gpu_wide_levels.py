"""V-cycles over levels of wide rows (a block per sixteen rows), against the oracle
at equal iterations: irregular matrices with and without hub rows, a wide level 0,
segments up to the block's sixteen rows and beyond them, level sizes that leave the
last block nearly empty, rows of one and of several steps of entries."""

import numpy as np
import pytest

import oracle
from gpu_helpers import setup, solve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,degree,hub,sweeps", [
    (400, 60.0, 0, 3), (1500, 12.0, 0, 3), (2500, 6.0, 900, 3), (6001, 9.0, 300, 1),
    (6001, 9.0, 0, 2), (6001, 9.0, 0, 4), (6001, 9.0, 300, 5), (20000, 12.0, 0, 3)])
def test_solve(n, degree, hub, sweeps, precision):
    from paper_2006_16147_amd import amg, inputs

    A = inputs.random_spd_graph(n, degree, seed=n, hub_degree=hub) if hub else \
        inputs.random_spd_graph(n, degree, seed=n)
    fp32 = precision == "fp32"
    h = setup(A, sweeps=sweeps, max_coarse=40, precision=amg.FP32 if fp32 else amg.FP64)
    ho = oracle.Hierarchy(A, sweeps=sweeps, max_coarse=40)
    assert h.sizes() == [ho.level_n(l) for l in range(ho.num_levels)]
    b = np.random.default_rng(1).uniform(-1, 1, A.n)
    st, info, x = solve(h, b, rtol=1e-8)
    assert st == 0 and info["converged"]
    xo, _ = ho.pcg(b, rtol=0.0, maxit=info["iterations"])
    # FP64: rounding of the sums; FP32: both within the stop test of the solution
    assert np.linalg.norm(x - xo) <= (1e-6 if fp32 else 1e-8) * np.linalg.norm(xo)
