"""Iterations are queued in chunks, and some while the host looks at the ones
before them: whatever the chunks, a solve stops at the first iteration that
meets the tolerance, or at maxit, with that iteration's x."""

import numpy as np
import pytest

from gpu_helpers import setup, solve

pytestmark = pytest.mark.gpu


def problem(name):
    from paper_2006_16147_amd import inputs

    A = {"grid": lambda: inputs.laplacian7(20), "tiny": lambda: inputs.laplacian7(6),
         "aniso": lambda: inputs.diffusion7(33, 0.3, 0.01, 1.0),
         "graph": lambda: inputs.random_spd_graph(3000, 6.0, seed=3)}[name]()
    return A, np.random.default_rng(7).uniform(-1, 1, A.n)


# hierarchies with iterations of few kernels, and with many: more sweeps, more levels
@pytest.mark.parametrize("name,params", [
    ("tiny", {}), ("grid", {}), ("grid", {"flags": 1}), ("aniso", {}), ("aniso", {"precision": 1}),
    ("graph", {"sweeps": 1}), ("grid", {"pre": 2, "post": 2}), ("grid", {"smooth_p": 1})])
def test_stops_where_it_should(name, params):
    from paper_2006_16147_amd import amg

    A, b = problem(name)
    h = setup(A, **params)
    x_at = {}
    for maxit in list(range(15)) + [17, 20]:
        st, info, x_at[maxit] = solve(h, b, rtol=0.0, maxit=maxit)
        assert st == amg.Status.NOT_CONVERGED and info["iterations"] == maxit
    for rtol in (0.9, 0.3, 1e-1, 1e-2, 1e-3, 9e-5, 1e-6, 1e-8):
        st, info, x = solve(h, b, rtol=rtol)
        assert st == amg.Status.OK and info["converged"] and info["rel_res_recursive"] <= rtol
        k = info["iterations"]
        if k in x_at:
            np.testing.assert_array_equal(x, x_at[k])
        if k > 0:  # not before
            st, info, x = solve(h, b, rtol=rtol, maxit=k - 1)
            assert st == amg.Status.NOT_CONVERGED and info["rel_res_recursive"] > rtol
        st, info, x = solve(h, b, rtol=rtol, maxit=k)
        assert st == amg.Status.OK and info["iterations"] == k
    h.close()
