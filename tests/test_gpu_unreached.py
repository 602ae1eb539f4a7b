"""Paths that the small cases of the other tests miss: edge correction beyond one chunk of
systems and beyond eight bin tuples per block of the matrix build, the 4PCF coupling of one
tuple of bins, and graph replays of a persistent gather."""
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


def test_several_chunks_equal_one(ctx):
    """6PCF lmax 3, 13 bins: 1,287 systems of 2,212 multiplets, 873 of which fit 32 GiB.
    A system's result does not depend on the chunk it is solved in: the same bits as from
    a call of 126 systems (9 bins), all in one chunk."""
    print("[unreached] chunks", flush=True)
    N, lmax = 6, 3
    n, nB, nS = encore.num_multiplets(N, lmax), encore.num_bin_tuples(N, 13), encore.num_bin_tuples(N, 9)
    rng = np.random.default_rng(6)
    R = rng.normal(0.0, 0.03, (n, nB))
    R[0] = rng.uniform(1.0, 3.0, nB)
    Nm = rng.normal(size=(n, nB))
    pick = np.concatenate([np.arange(0, 42), np.arange(852, 894), np.arange(nB - 42, nB)])   # around the border at 873
    assert len(pick) == nS
    z = encore.edge_correct(ctx, N, lmax, 13, Nm, R)
    part = encore.edge_correct(ctx, N, lmax, 9, np.ascontiguousarray(Nm[:, pick]), np.ascontiguousarray(R[:, pick]))
    assert np.array_equal(z[:, pick], part)
    assert np.all(np.isfinite(z))


def test_more_than_2400_multiplets(ctx):
    """5PCF lmax 5, all parities: 2,666 multiplets, four bin tuples per block of the matrix
    build.  Row L = 0 in closed form: M[0][L''] = (4 pi)^-2 f_L''; the matrix is linear in
    the window; the solution solves the device's own systems."""
    print("[unreached] 2666 multiplets", flush=True)
    N, lmax, nbins = 5, 5, 6
    n, nB = encore.num_multiplets(N, lmax, True), encore.num_bin_tuples(N, nbins)
    assert n == 2666 and nB == 15
    rng = np.random.default_rng(8)
    R = rng.normal(0.0, 0.03, (n, nB))
    R[0] = 2.0
    R[1:, 14] = R[1:, 3] + R[1:, 8]
    Nm = rng.normal(size=(n, nB))
    z, M, bad = encore.edge_correct(ctx, N, lmax, nbins, Nm, R, allparity=True, return_coupling=True)
    assert bad == 0
    c = (4.0 * np.pi) ** -2
    for b in range(nB):
        assert np.max(np.abs(M[b, 0] - c * R[:, b] / R[0, b])) <= 1e-15
        A = M[b].T
        r = A @ z[:, b] - Nm[:, b] / R[0, b]
        # backward stable: residual of the size of n eps |A| |z|
        assert np.max(np.abs(r)) <= 1e-13 * np.max(np.abs(A) @ np.abs(z[:, b]))
    lin = M[3] + M[8] - c * np.eye(n) - M[14]
    assert np.max(np.abs(lin)) <= 1e-13 * np.max(np.abs(M[14]))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_couple4_three_bins(ctx, precision):
    """One tuple of bins and enough tuples of (l, m) for the 4PCF's own kernel (lmax 9)."""
    print("[unreached] couple4 3 bins %s" % precision, flush=True)
    rng = np.random.default_rng(12)
    pos, w = rng.uniform(0.0, 60.0, (150, 3)), rng.uniform(-0.5, 1.5, 150)
    edges = np.linspace(4.0, 28.0, 4)
    lmax = 9
    lam, l, m, coef = encore.coupling_terms(4, lmax)
    assert len({tuple(x) for x in np.concatenate([l, m], axis=1)}) >= 8192
    prim = np.arange(2, 150, 5)
    zo, za = oracle.zeta(pos, w, 4, lmax, edges, box=60.0, primaries=prim, return_abs=True)
    with encore.build_grid(ctx, pos, w, r_max=edges[-1], box=60.0) as g:
        zg = encore.npcf(ctx, g, 4, lmax, edges, precision=precision, primaries=prim)
    bars.check(zg, zo, za, precision, "3 bins")


def test_graph_replays_persistent_gather(ctx):
    """A recorded plan whose gather takes the persistent grid (its queues are cleared in
    the graph): every replay is the eager result, with eager work between them."""
    print("[unreached] graph", flush=True)
    rng = np.random.default_rng(13)
    n = 90_000
    pos, w = rng.uniform(0.0, 300.0, (n, 3)), rng.uniform(0.5, 1.5, n)
    edges = np.linspace(4.0, 16.0, 7)       # 270,000 items of two bins
    with encore.build_grid(ctx, pos, w, r_max=edges[-1], box=300.0) as g, \
            encore.build_grid(ctx, pos[:5000], w[:5000], r_max=edges[-1], box=300.0) as other:
        for precision in ("splitbf16", "fp32"):
            eager = encore.npcf(ctx, g, 3, 3, edges, precision=precision)
            with encore.Plan(ctx, g, 3, 3, edges, precision=precision) as p:
                for _ in range(4):
                    assert np.array_equal(p.execute(), eager), precision
                    encore.npcf(ctx, other, 4, 2, edges, precision=precision)
                    ctx.last_timings()
