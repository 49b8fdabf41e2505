"""The rule for levels of wide rows on both sides of its row limit: up to 32768
rows from 32 stored entries per row, above from 64. One V-cycle against the
oracle's on the same vector."""

import numpy as np
import pytest

import oracle
from gpu_helpers import setup, to_dev

pytestmark = pytest.mark.gpu


# (slices of 64 rows are padded to their longest row: 34 to 62 entries stored
# per row at degrees 21 and 45, 80 at degree 60)
@pytest.mark.parametrize("n,degree", [(32768, 21.0), (32768, 45.0), (32769, 45.0), (32769, 60.0),
                                      (40000, 60.0)])
def test_application(n, degree):
    import torch

    from paper_2006_16147_amd import amg, inputs

    A = inputs.random_spd_graph(n, degree, seed=n)
    width = np.diff(A.row_ptr)
    pad = -n % 64
    stored = np.concatenate([width, np.zeros(pad, dtype=width.dtype)]).reshape(-1, 64).max(1).sum()
    mean = stored * 64 / n
    assert (32 <= mean < 64) if degree < 60 else mean >= 64
    h = setup(A, max_levels=3, max_coarse=4096, sweeps=2)
    ho = oracle.Hierarchy(A, max_levels=3, max_coarse=4096, sweeps=2)
    assert h.sizes() == ho.sizes()
    r = np.random.default_rng(3).uniform(-1, 1, n)
    z = torch.zeros(n, dtype=torch.float64, device="cuda")
    amg.amg_vcycle_apply(h, to_dev(r), z)
    zo = ho.vcycle(r)
    np.testing.assert_allclose(z.cpu().numpy(), zo, rtol=0, atol=1e-10 * np.abs(zo).max())
    h.close()
