"""CG on a matrix that is not positive definite: the solve ends in a breakdown,
and the x it returns is the iterate before it, the same on every call."""

import numpy as np
import pytest

from gpu_helpers import setup, solve

pytestmark = pytest.mark.gpu


def indefinite(N, weight):
    """The 7-point Laplacian beside a pair of vertices with the eigenvalues 3 and
    -1; the pair's aggregate holds only the first, so that the setup accepts it.
    weight: of the second's eigenvector in the right-hand side."""
    from paper_2006_16147_amd import inputs

    A = inputs.laplacian7(N)
    n = A.n
    rp = np.concatenate([A.row_ptr, A.row_ptr[-1] + np.array([2, 4])])
    col = np.concatenate([A.col, [n, n + 1, n, n + 1]])
    val = np.concatenate([A.val, [1.0, 2.0, 2.0, 1.0]])
    b = np.random.default_rng(N).uniform(-1, 1, n + 2)
    b[n:] = weight, -weight
    return inputs.Csr(n + 2, rp, col, val), b


# systems whose kernels sum the scalars themselves (the last: in about as many
# blocks as there may be), and one above them
@pytest.mark.parametrize("pre", [1, 2])
@pytest.mark.parametrize("N", [7, 20, 50, 56])
def test_breakdown_returns_the_iterate_before_it(N, pre):
    from paper_2006_16147_amd import amg

    A, b = indefinite(N, 1e-3)
    h = setup(A, pre=pre, post=pre)
    for flags in (0, amg.FLAG_NO_GRAPH):
        k = setup(A, pre=pre, post=pre, flags=flags) if flags else h
        st, info, x = solve(k, b, rtol=1e-12, maxit=500)
        assert st == amg.Status.ERR_BREAKDOWN, (st, info)
        last = info["iterations"]
        assert last > 1
        st, info, want = solve(k, b, rtol=0.0, maxit=last)
        assert st == amg.Status.NOT_CONVERGED and info["iterations"] == last
        np.testing.assert_array_equal(x, want)
        for _ in range(10):
            st, info, x = solve(k, b, rtol=1e-12, maxit=500)
            assert st == amg.Status.ERR_BREAKDOWN and info["iterations"] == last
            np.testing.assert_array_equal(x, want)
    h.close()
