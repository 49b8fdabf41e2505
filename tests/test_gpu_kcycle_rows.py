"""K-cycle levels of short and of long rows take different kernels: irregular
matrices and grids whose levels lie on both sides of that rule, with last levels
that go into the one-block step and that do not, against the oracle."""

import numpy as np
import pytest

import oracle
from gpu_helpers import setup, to_dev

pytestmark = pytest.mark.gpu


def operator(name):
    from paper_2006_16147_amd import inputs

    kind, *sizes = name.split(":")
    if kind == "graph":
        return inputs.random_spd_graph(int(sizes[0]), float(sizes[1]), seed=2)
    if kind == "blocks":
        N = int(sizes[0])
        ex, ey = inputs.block_log_uniform_eps(N, 8, np.random.default_rng(3))
        return inputs.diffusion7(N, ex, ey, 1.0)
    return inputs.laplacian7(int(sizes[0]))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", ["graph:2000:5", "graph:3000:4", "graph:4000:5", "graph:5000:6",
                                  "graph:10000:9", "graph:9000:14", "blocks:32", "blocks:40",
                                  "poisson:24"])
def test_application(name, precision):
    import torch

    from paper_2006_16147_amd import amg

    A = operator(name)
    h = setup(A, cycle=amg.CYCLE_K, precision=amg.FP32 if precision == "fp32" else amg.FP64)
    ho = oracle.Hierarchy(A)
    assert h.sizes() == ho.sizes()
    r = np.random.default_rng(7).uniform(-1, 1, A.n)
    z = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    amg.amg_vcycle_apply(h, to_dev(r), z)
    zo = ho.kcycle(r)
    # rounding of the sums, in the hierarchy's precision
    tol = 1e-10 if precision == "fp64" else 1e-4
    np.testing.assert_allclose(z.cpu().numpy(), zo, rtol=0, atol=tol * np.abs(zo).max())
    h.close()
