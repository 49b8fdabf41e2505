"""K-cycle levels on both sides of the sizes where the prolongation moves into
the post-sweep, r1 = b - s1 v1 into the down step and the level above the
coarsest into one block: one application against the oracle's on the same vector."""

import numpy as np
import pytest

import oracle
from gpu_helpers import setup, to_dev

pytestmark = pytest.mark.gpu


def operator(name):
    from paper_2006_16147_amd import inputs

    if name.startswith("poisson"):
        return inputs.laplacian7(int(name[7:]))
    if name.startswith("aniso"):
        return inputs.diffusion7(int(name[5:]), 0.3, 0.01, 1.0)
    return inputs.random_spd_graph(int(name[5:]), 6.0, seed=3, hub_degree=200)


# poisson22: one block with two rows per thread and two passes over A_L^-1;
# poisson45: the same below two levels that prolong in the post-sweep; poisson104: a level
# of more than 131072 rows, with the separate kernels; post = 2 or pre = 2: one of the
# two without the other; sweeps: aggregates of up to 4 and 32
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name,params", [
    ("poisson22", {}), ("poisson45", {}), ("poisson104", {}),
    ("aniso30", {"pre": 1, "post": 2}), ("aniso30", {"pre": 2, "post": 1}),
    ("graph6000", {"sweeps": 2}), ("poisson40", {"sweeps": 5, "max_coarse": 30})])
def test_application(name, params, precision):
    import torch

    from paper_2006_16147_amd import amg

    A = operator(name)
    sm = {k: v for k, v in params.items() if k in ("pre", "post")}
    hp = {k: v for k, v in params.items() if k not in sm}
    h = setup(A, cycle=amg.CYCLE_K, precision=amg.FP32 if precision == "fp32" else amg.FP64,
              **params)
    ho = oracle.Hierarchy(A, **hp)
    assert h.sizes() == [ho.level_n(l) for l in range(ho.num_levels)]
    r = np.random.default_rng(7).uniform(-1, 1, A.n)
    z = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    amg.amg_vcycle_apply(h, to_dev(r), z)
    zo = ho.kcycle(r, **sm)
    tol = 1e-10 if precision == "fp64" else 1e-4
    np.testing.assert_allclose(z.cpu().numpy(), zo, rtol=0, atol=tol * np.abs(zo).max())
