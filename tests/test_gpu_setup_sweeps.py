"""Pairwise sweeps of the setup at the sizes where their kernels split: vertices
per matching block, lanes per row, listed long rows; the hierarchy bit for bit
against the oracle, and the matching's rounds against a synchronous model."""

import numpy as np
import pytest

import oracle
from gpu_helpers import assert_same_hierarchy, setup, setup_status

pytestmark = pytest.mark.gpu


def path_matrix(weights):
    """A path with the given off-diagonal magnitudes, as CSR."""
    from paper_2006_16147_amd import inputs

    n = len(weights) + 1
    rows, cols, vals = [], [], []
    for i in range(n):
        s = 0.5
        left = weights[i - 1] if i > 0 else 0.0
        right = weights[i] if i < n - 1 else 0.0
        for j, a in ((i - 1, -left), (i, s + left + right), (i + 1, -right)):
            if 0 <= j < n:
                rows.append(i)
                cols.append(j)
                vals.append(a)
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))])
    return inputs.Csr(n, rp, np.array(cols), np.array(vals))


def synchronous_rounds(A, w):
    """Rounds in which some vertex still proposes after the first proposals."""
    d = np.array([A.val[A.row_ptr[i]:A.row_ptr[i + 1]][
        A.col[A.row_ptr[i]:A.row_ptr[i + 1]] == i][0] for i in range(A.n)])
    lists = []
    for i in range(A.n):
        es = []
        for k in range(A.row_ptr[i], A.row_ptr[i + 1]):
            j = int(A.col[k])
            if j != i:
                lo, hi = min(i, j), max(i, j)
                c = 1.0 - (((2.0 * A.val[k]) * w[lo]) * w[hi]) / (
                    (d[lo] * w[lo]) * w[lo] + (d[hi] * w[hi]) * w[hi])
                es.append((-c, lo, hi, j))
        lists.append([e[3] for e in sorted(es)])
    taken = np.zeros(A.n, dtype=bool)
    rounds = -1
    while True:
        prop = [next((j for j in lists[i] if not taken[j]), -1) if not taken[i] else -1
                for i in range(A.n)]
        for i in range(A.n):
            if not taken[i] and prop[i] < 0:
                taken[i] = True
        if all(p < 0 for p in prop):
            return max(rounds, 0)
        rounds += 1
        for i in range(A.n):
            if prop[i] >= 0 and prop[prop[i]] == i:
                taken[i] = True


@pytest.mark.parametrize("n", [2, 3, 511, 512, 513, 1537])
@pytest.mark.parametrize("order", ["equal", "rising", "falling"])
def test_path(n, order):
    # rising weights: the chain of dependent matches runs from the last vertex back
    weights = {"equal": np.ones(n - 1), "rising": 1.0 + np.arange(n - 1),
               "falling": 1.0 * n - np.arange(n - 1)}[order]
    A = path_matrix(weights)
    h = setup(A, max_coarse=1)
    ho = oracle.Hierarchy(A, max_coarse=1)
    assert_same_hierarchy(h, ho)
    h.close()
    if n > 1:
        h = setup(A, max_coarse=1, sweeps=1)
        assert h.matching_rounds(0) == synchronous_rounds(A, np.ones(n))
        h.close()


@pytest.mark.parametrize("n,degree,hub", [
    (600, 1.5, 0), (700, 7.0, 17), (900, 8.5, 33), (1025, 16.0, 65), (800, 31.0, 129),
    (513, 70.0, 0), (1500, 6.0, 700), (2100, 6.0, 1400)])
def test_row_lengths(n, degree, hub):
    from paper_2006_16147_amd import inputs

    A = inputs.random_spd_graph(n, degree, seed=n, hub_degree=hub)
    h = setup(A, max_coarse=40)
    ho = oracle.Hierarchy(A, max_coarse=40)
    assert_same_hierarchy(h, ho)
    h.close()
    if n <= 1025:
        h = setup(A, max_coarse=40, sweeps=1)
        assert h.matching_rounds(0) == synchronous_rounds(A, np.ones(n))
        h.close()


def test_row_too_long_is_refused():
    from paper_2006_16147_amd import amg, inputs

    A = inputs.random_spd_graph(3000, 4.0, seed=1, hub_degree=2500)
    st, h = setup_status(A)
    assert st == amg.Status.ERR_ARG and h is None


@pytest.mark.parametrize("n,degree,hub,sweeps", [
    (900, 3.0, 0, 3), (3000, 6.0, 250, 3), (800, 60.0, 0, 3), (2000, 12.0, 0, 2),
    (12000, 70.0, 0, 8)])  # the last: columns of Pbar longer than a block sorts in LDS
def test_smoothed_products(n, degree, hub, sweeps):
    from paper_2006_16147_amd import inputs

    A = inputs.random_spd_graph(n, degree, seed=n, hub_degree=hub)
    h = setup(A, smooth_p=1, max_coarse=60, sweeps=sweeps)
    ho = oracle.Hierarchy(A, smooth=True, max_coarse=60, sweeps=sweeps)
    assert ho.ok
    assert_same_hierarchy(h, ho)
    for l in range(ho.num_levels - 1):
        (rp, ci, val), om = h.prolongator(l)
        rpo, cio, valo = ho.pbar(l)
        assert om == ho.omega(l)
        np.testing.assert_array_equal(rp, rpo)
        np.testing.assert_array_equal(ci, cio)
        np.testing.assert_array_equal(val.view(np.uint64), valo.view(np.uint64))
    h.close()
