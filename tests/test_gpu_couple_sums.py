"""The FP64 4PCF coupling sums tiles of primaries before it adds them to the running
sum (10 radial bins): small terms after a large one are not lost one by one.

One primary carries a weight that makes its term 1.5 * 2^52 units; 63 primaries of
another cluster, out of reach of it, follow with terms of at most 0.49 units, each of
which would be rounded away if it were added to the running sum by itself (their sum
is more than 20 units).  At lmax 5 a tile holds 9 primaries, so the sum over tiles is
off by at most half a unit for each of the 7 later tiles, by the first tile's 8 terms
(3.9 units) and by 4 units of rounding in the products and the contraction: 12 units.
The exact value comes from the device's own coefficients in rational arithmetic.
"""
from fractions import Fraction

import numpy as np
import pytest

from paper_2105_08722_amd import encore

pytestmark = pytest.mark.gpu


def test_small_terms_after_a_large_one():
    print("[couple-sums] lmax 5, 10 bins, fp64", flush=True)
    rng = np.random.default_rng(5)
    lmax, nbins = 5, 10
    edges = np.linspace(2.0, 22.0, nbins + 1)
    far = rng.uniform(0.0, 30.0, (4000, 3)) + 100.0
    near = rng.uniform(-14.0, 14.0, (300, 3))
    pos = np.concatenate([[[0.0, 0.0, 0.0]], near, far])
    w = np.ones(len(pos))
    b = (2, 5, 8)
    tuples = [(i, j, k) for i in range(nbins) for j in range(i + 1, nbins) for k in range(j + 1, nbins)]
    assert len(tuples) == encore.num_bin_tuples(4, nbins)
    with encore.Context(0) as ctx:
        with encore.build_grid(ctx, pos, w, r_max=edges[-1]) as g:
            cand = np.concatenate([[0], np.arange(301, len(pos))])
            a = encore.debug_alm(ctx, g, lmax, edges, cand, "fp64")[:, list(b), 0].real     # l = m = 0
        keep = np.concatenate([[0], 1 + np.argsort(-a[1:].prod(axis=1))[:63]])   # the largest terms
        prim, a = cand[keep], a[keep]
        assert a.min() > 0.0
        unit = float(a[1:].prod(axis=1).max()) / 0.49
        w[0] = 1.5 * 2.0 ** 52 * unit / float(a[0].prod())
        with encore.build_grid(ctx, pos, w, r_max=edges[-1]) as g:
            z = encore.npcf(ctx, g, 4, lmax, edges, precision="fp64", primaries=prim)[0, tuples.index(b)]
    terms = [Fraction(float(w[i])) * Fraction(float(a[k, 0])) * Fraction(float(a[k, 1])) * Fraction(float(a[k, 2]))
             for k, i in enumerate(prim)]
    assert sum(terms[1:]) > 20 * Fraction(unit)
    lam, l, m, coef = encore.coupling_terms(4, lmax)
    c = [float(coef[t]) for t in range(len(lam)) if lam[t] == 0]
    assert len(c) == 1
    want = Fraction(c[0]) * sum(terms)
    off = abs(Fraction(float(z)) - want) / (Fraction(abs(c[0])) * Fraction(unit))
    print("[couple-sums] off by %.2f units" % float(off), flush=True)
    assert off <= 12
