"""The block solve where residual and restriction are one kernel and z is formed
in the prolongation: column blocks that take it, with full and ragged tiles, one
and four passes per block, against narrow blocks (k odd) that take the separate
kernels, and against the oracle."""

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


def block(h, B, its):
    import torch

    from paper_2006_16147_amd import amg

    Bd = to_dev(np.ascontiguousarray(B))
    X = torch.zeros_like(Bd)
    st, infos = amg.amg_pcg_solve_batch(h, Bd, X, rtol=0.0, maxit=its, raise_on_error=False)
    assert st == amg.Status.NOT_CONVERGED and all(i["iterations"] == its for i in infos)
    return X.cpu().numpy()


# sweeps 1: segments of two, 5: up to 32 rows, more than a block's pass holds at
# wide tiles; 13^3 and the graph: last blocks nearly empty; 42^3 with k = 64 and 48^3
# with k = 36: four passes per block on level 0 and one below
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name,k,sweeps", [
    ("poisson13", 4, 3), ("poisson13", 12, 1), ("poisson13", 36, 5), ("aniso16", 64, 2),
    ("aniso16", 260, 5), ("graph2500", 8, 3), ("graph2500", 20, 4), ("poisson42", 64, 3),
    ("aniso48", 36, 3)])
def test_down_step(name, k, sweeps, precision):
    from paper_2006_16147_amd import amg

    A = operator(name)
    fp32 = precision == "fp32"
    h = setup(A, sweeps=sweeps, max_coarse=40, precision=amg.FP32 if fp32 else amg.FP64)
    B = np.random.default_rng(k).uniform(-1, 1, (A.n, k))
    X = block(h, B, 5)
    # five iterations apart only in the grouping of the dot products: rounding of
    # the FP64 scalars, and the FP32 rounding of r that follows it
    tol = 1e-8 if fp32 else 1e-11
    for cols in (slice(0, 3), slice(k - 3, k)):
        Y = block(h, B[:, cols], 5)
        err = np.linalg.norm(X[:, cols] - Y, axis=0) / np.linalg.norm(Y, axis=0)
        assert (err <= tol).all(), err
    if not fp32 and A.n < 5000:
        xo, _ = oracle.Hierarchy(A, sweeps=sweeps, max_coarse=40).pcg(B[:, k - 1], rtol=0.0, maxit=5)
        assert np.linalg.norm(X[:, k - 1] - xo) <= 1e-10 * np.linalg.norm(xo)
