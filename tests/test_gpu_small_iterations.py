"""CG iterations in the forms that small systems take (scalars summed by the
kernels that use them, p = z + beta p inside the product with A), on both sides
of the sizes where each form begins, against the oracle at equal iterations."""

import numpy as np
import pytest

import oracle
from gpu_helpers import setup, solve

pytestmark = pytest.mark.gpu


def operator(name):
    from paper_2006_16147_amd import inputs

    if name.startswith("poisson"):
        return inputs.laplacian7(int(name[7:]))
    if name.startswith("aniso"):
        return inputs.diffusion7(int(name[5:]), 0.3, 0.01, 1.0)
    return inputs.random_spd_graph(int(name[5:]), 6.0, seed=3, hub_degree=200)


@pytest.mark.parametrize("smoothed", [False, True])
@pytest.mark.parametrize("sweeps", [1, 2])
@pytest.mark.parametrize("name", ["poisson7", "poisson13", "aniso16", "graph2500"])
def test_folded(name, sweeps, smoothed):
    A = operator(name)
    h = setup(A, pre=sweeps, post=sweeps, smooth_p=int(smoothed))
    ho = oracle.Hierarchy(A, smooth=smoothed)
    rng = np.random.default_rng(1)
    b, x0 = rng.uniform(-1, 1, A.n), rng.uniform(-1, 1, A.n)
    for start in (np.zeros(A.n), x0):
        st, info, x = solve(h, b, start, rtol=1e-8)
        assert st == 0 and info["converged"]
        xo, _ = ho.pcg(b, x0=start, rtol=0.0, maxit=info["iterations"], pre=sweeps, post=sweeps)
        assert np.linalg.norm(x - xo) <= 1e-8 * np.linalg.norm(xo)
    # cut short, and nothing to do
    st, info, x = solve(h, b, rtol=0.0, maxit=3)
    assert st == 8 and info["iterations"] == 3
    xo, _ = ho.pcg(b, rtol=0.0, maxit=3, pre=sweeps, post=sweeps)
    assert np.linalg.norm(x - xo) <= 1e-10 * np.linalg.norm(xo)
    st, info, x = solve(h, np.zeros(A.n), x0)
    assert st == 0 and info["iterations"] == 0 and not x.any()
    st, info, x = solve(h, b, rtol=1e-8, maxit=0)
    assert st == 8 and info["iterations"] == 0 and not x.any()
    h.close()


# 131072 rows: the last with folded scalars; 2^20: the last with one sum for
# the stop test and beta
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", ["poisson50", "poisson51", "poisson101", "poisson102"])
def test_sizes_where_the_forms_change(name, precision):
    from paper_2006_16147_amd import amg

    A = operator(name)
    h = setup(A, precision=amg.FP32 if precision == "fp32" else amg.FP64)
    ho = oracle.Hierarchy(A)
    b = np.random.default_rng(2).uniform(-1, 1, A.n)
    st, info, x = solve(h, b, rtol=1e-8)
    assert st == 0 and info["converged"] and info["rel_res_true"] <= 1.01e-8
    xo, _ = ho.pcg(b, rtol=0.0, maxit=info["iterations"])
    assert np.linalg.norm(x - xo) <= 1e-8 * np.linalg.norm(xo)
    h.close()
