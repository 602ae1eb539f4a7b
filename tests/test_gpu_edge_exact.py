"""Rounding of the edge solve: its error against the solution in extended precision of
the device's own systems, over 330 systems of 65 multiplets (a panel and one column)
and 40 of 204 (two outer blocks), windows with 3% multiplets.

The bounds are what an elimination reaches whose updates are summed over 32 columns
before they are subtracted, rms over systems, in units of 2^-53 of the solution's
norm: 3.8 and 6.1, each with 4 standard errors of the sample (0.14 and 0.3).
"""
import numpy as np
import pytest
from scipy.linalg import lu_factor, lu_solve

from paper_2105_08722_amd import encore

pytestmark = pytest.mark.gpu


def _exact(A, b):
    """A x = b by iterative refinement with residuals in extended precision."""
    lu, Al, bl = lu_factor(A), A.astype(np.longdouble), b.astype(np.longdouble)
    x = lu_solve(lu, b).astype(np.longdouble)
    for _ in range(5):
        x = x + lu_solve(lu, (bl - Al @ x).astype(np.float64))
    return x


@pytest.mark.parametrize("N,lmax,nbins,allp,seeds,systems,bound", [(4, 4, 11, True, 2, 165, 3.94),
                                                                   (5, 3, 9, False, 1, 40, 6.4)])
def test_solve_rounding(N, lmax, nbins, allp, seeds, systems, bound):
    n, nB = encore.num_multiplets(N, lmax, allp), encore.num_bin_tuples(N, nbins)
    print("[edge-exact] N %d lmax %d n %d" % (N, lmax, n), flush=True)
    e = []
    with encore.Context(0) as ctx:
        for s in range(seeds):
            rng = np.random.default_rng(1000 + n + 77 * s)
            R = rng.normal(0.0, 0.03, (n, nB))
            R[0] = rng.uniform(1.0, 3.0, nB)
            D = rng.normal(size=(n, nB))
            z, M, bad = encore.edge_correct(ctx, N, lmax, nbins, D, R, allparity=allp, return_coupling=True)
            assert bad == 0
            for b in range(systems):
                x = _exact(M[b].T.copy(), D[:, b] / R[0, b])
                e.append(float(np.linalg.norm((z[:, b] - x).astype(np.float64)) / np.linalg.norm(x.astype(np.float64))))
    rms = float(np.sqrt(np.mean(np.square(e)))) * 2.0 ** 53
    print("[edge-exact] rms %.2f units" % rms, flush=True)
    assert rms <= bound
