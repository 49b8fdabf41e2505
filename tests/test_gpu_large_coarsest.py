"""Coarsest levels above the size whose factorization fits in LDS: Cholesky by
panels (sizes around a panel, a tile and a block of rows) against a dense solve,
the many-block coarsest product inside a cycle against the oracle, and a matrix that
is not positive definite from a given column on."""

import numpy as np
import pytest

import oracle
from gpu_helpers import setup, setup_status, solve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [201, 223, 224, 225, 256, 257, 480, 545, 1031])
def test_one_level(n):
    from paper_2006_16147_amd import inputs

    A = inputs.random_spd_graph(n, 12.0, seed=n)
    h = setup(A, max_coarse=n)
    assert h.sizes() == [n]
    b = np.random.default_rng(n).uniform(-1, 1, n)
    st, info, x = solve(h, b, rtol=1e-12)
    assert st == 0 and info["iterations"] <= 2
    # diagonally dominant: a condition number of at most a few hundred
    xd = np.linalg.solve(A.to_dense(), b)
    assert np.linalg.norm(x - xd) <= 1e-11 * np.linalg.norm(xd)


@pytest.mark.parametrize("cycle", ["V", "K"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_cycle(precision, cycle):
    from paper_2006_16147_amd import amg, inputs

    A = inputs.random_spd_graph(9000, 7.0, seed=5)
    fp32 = precision == "fp32"
    h = setup(A, max_coarse=1400, precision=amg.FP32 if fp32 else amg.FP64,
              cycle=amg.CYCLE_K if cycle == "K" else amg.CYCLE_V)
    ho = oracle.Hierarchy(A, max_coarse=1400)
    assert h.sizes() == [ho.level_n(l) for l in range(ho.num_levels)] and h.sizes()[-1] > 256
    b = np.random.default_rng(1).uniform(-1, 1, A.n)
    st, info, x = solve(h, b, rtol=1e-8)
    assert st == 0 and info["converged"]
    pcg = ho.fcg if cycle == "K" else ho.pcg
    xo = pcg(b, rtol=0.0, maxit=info["iterations"])[0]
    assert np.linalg.norm(x - xo) <= (1e-6 if fp32 else 1e-8) * np.linalg.norm(xo)


@pytest.mark.parametrize("k", [0, 31, 32, 150, 298])
def test_not_positive_definite(k):
    from paper_2006_16147_amd import amg, inputs

    D = inputs.random_spd_graph(300, 8.0, seed=2).to_dense()
    D[k, k + 1] = D[k + 1, k] = -2.0 * np.sqrt(D[k, k] * D[k + 1, k + 1])
    row, col = np.nonzero(D)
    ptr = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=300))])
    A = inputs.Csr(300, ptr, col, D[row, col])
    assert setup_status(A, max_coarse=300)[0] == amg.Status.ERR_NOT_SPD
