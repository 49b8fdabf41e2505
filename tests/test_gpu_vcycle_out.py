"""amg_vcycle_apply where the last post-sweep stores z in the caller's numbering
(V-cycle of more than one level) and where a permutation follows (one level):
against the oracle, into a block of its own and over r."""

import numpy as np
import pytest

import oracle
from gpu_helpers import setup, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name,params", [
    ("poisson5", {}), ("poisson20", {}), ("poisson20", {"post": 3}), ("poisson17", {"smooth_p": 1}),
    ("aniso21", {}), ("graph3000", {"pre": 2}), ("graph3000", {"smooth_p": 1})])
def test_apply(name, params, precision):
    import torch

    from paper_2006_16147_amd import amg, inputs

    N = int(name.lstrip("poisnagrh"))
    A = (inputs.laplacian7(N) if name.startswith("poisson") else
         inputs.diffusion7(N, 0.3, 0.01, 1.0) if name.startswith("aniso") else
         inputs.random_spd_graph(N, 7.0, seed=4, hub_degree=120))
    h = setup(A, precision=amg.FP32 if precision == "fp32" else amg.FP64, **params)
    ho = oracle.Hierarchy(A, smooth=bool(params.get("smooth_p")))
    r = np.random.default_rng(7).uniform(-1, 1, A.n)
    zo = ho.vcycle(r, pre=params.get("pre", 1), post=params.get("post", 1))
    tol = 1e-12 if precision == "fp64" else 1e-4
    rd = to_dev(r)
    z = torch.full((A.n,), float("nan"), dtype=torch.float64, device="cuda")
    amg.amg_vcycle_apply(h, rd, z)
    np.testing.assert_allclose(z.cpu().numpy(), zo, rtol=0, atol=tol * np.abs(zo).max())
    first = z.clone()
    amg.amg_vcycle_apply(h, rd, rd)
    assert torch.equal(rd, first)
