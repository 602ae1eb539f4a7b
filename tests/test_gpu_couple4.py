"""The 4PCF coupling over first bins (k_couple4) against the oracle at the bin counts
and degrees where its dispatch changes: 3 bins (one tuple of bins) to 13 (the general
kernel again), FP64 and FP32, both parities, and primaries that do not fill a tile or a
split.  Bars: tests/parity_bars.py (FP64 1e-10 of max|Z|; FP32 1e-6 and the conditioning).
"""
import numpy as np
import pytest

import oracle
import parity_bars as bars
from paper_2105_08722_amd import encore

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = encore.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nbins,lmax,allp", [(3, 5, False), (5, 4, True), (7, 3, False), (7, 4, False), (8, 4, False),
                                             (9, 3, True), (10, 2, False), (11, 3, False), (12, 4, False),
                                             (13, 3, False)])
def test_zeta_over_bin_counts(ctx, nbins, lmax, allp, precision):
    print("[couple4] nbins %d lmax %d allparity %s %s" % (nbins, lmax, allp, precision), flush=True)
    rng = np.random.default_rng(100 * nbins + lmax)
    n = 331
    pos = rng.uniform(0.0, 60.0, (n, 3))
    w = rng.uniform(-0.5, 1.5, n)
    edges = np.linspace(2.0, 29.0, nbins + 1)
    parity = "all" if allp else "even"
    for prim in (None, np.arange(3, n, 7)):
        zo, za = oracle.zeta(pos, w, 4, lmax, edges, box=60.0, parity=parity, primaries=prim, return_abs=True)
        with encore.build_grid(ctx, pos, w, r_max=edges[-1], box=60.0) as g:
            zg = encore.npcf(ctx, g, 4, lmax, edges, precision=precision, allparity=allp, primaries=prim)
        bars.check(zg, zo, za, precision, "nbins %d" % nbins)
