"""Pairwise Galerkin rows that gather more than 2048 fine entries from two
matched rows of at most 2048 each: refused whichever sweep of a level forms
them, in plain and in smoothed set-ups; exactly 2048 are accepted."""

import numpy as np
import pytest

import oracle
from gpu_helpers import assert_same_hierarchy, setup, setup_status

pytestmark = pytest.mark.gpu


def hub_pairs(leaves, chain=600):
    """len(leaves) hubs (a power of two), hub i with leaves[i] neighbours of its
    own, joined by ever weaker edges so that sweep k matches the aggregates of
    2^k hubs with each other and leaves their neighbours alone; and a chain of
    vertices beside them, in which every sweep matches something."""
    from paper_2006_16147_amd import inputs

    m, n = len(leaves), len(leaves) + sum(leaves) + chain
    edges, at = [], m
    for i, k in enumerate(leaves):
        edges += [(i, at + q, 0.01) for q in range(k)]
        at += k
    edges += [(i, i + 1, 1.0) for i in range(at, n - 1)]
    step, a = 1, 1000.0
    while step < m:
        edges += [(i, i + step, a) for i in range(0, m, 2 * step)]
        step, a = 2 * step, a / 10.0
    diag = np.full(n, 0.5)
    rows, cols, vals = list(range(n)), list(range(n)), []
    for i, j, a in edges:
        diag[i] += a
        diag[j] += a
    vals += list(diag)
    for i, j, a in edges:
        rows += [i, j]
        cols += [j, i]
        vals += [-a, -a]
    order = np.lexsort((cols, rows))
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))])
    return inputs.Csr(n, rp, np.array(cols)[order], np.array(vals)[order])


@pytest.mark.parametrize("smooth_p", [0, 1])
@pytest.mark.parametrize("leaves,sweeps", [
    ([1100] * 2, 1), ([1100] * 2, 2), ([1100] * 2, 3),  # formed by the first sweep
    ([550] * 4, 2), ([550] * 4, 3),                     # by the second
    ([275] * 8, 3), ([275] * 8, 8),                     # by the third
    ([2039, 9], 3)])                                    # a long row and a short one
def test_refused_in_every_sweep(leaves, sweeps, smooth_p):
    from paper_2006_16147_amd import amg

    # (two levels: the next one's own limits do not come into it)
    st, h = setup_status(hub_pairs(leaves), sweeps=sweeps, smooth_p=smooth_p, max_levels=2)
    assert st == amg.Status.ERR_ARG and h is None


def test_most_entries_accepted():
    from paper_2006_16147_amd import amg

    # two rows of 1024 entries; one more is refused
    A = hub_pairs([1022, 1022], chain=0)
    h = setup(A, sweeps=1, max_levels=2)
    ho = oracle.Hierarchy(A, sweeps=1, max_levels=2)
    assert ho.sizes() == [2046, 2045]
    assert_same_hierarchy(h, ho)
    h.close()
    st, h = setup_status(hub_pairs([1023, 1022], chain=0), sweeps=1, max_levels=2)
    assert st == amg.Status.ERR_ARG and h is None
