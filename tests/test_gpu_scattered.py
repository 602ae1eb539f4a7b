"""Primaries in any order over a catalog beyond the caches take more bins per work item
in the plain FP32 gather, at lmax 0 to 4: their coefficients against the oracle at bin
counts around the group sizes, and the same bits alone, in a batch beside a job that
takes two bins, over several slices and without allocation.

Tolerance of the coefficients: plain FP32 sums, at most 200 pairs per bin, 4 additions
per lane and 6 of the lane tree, and a term's own rounding (about 10 operations), each
6e-8 of a sum that is at most sqrt(2 lmax + 1) times the monopole's: 20 * 6e-8 * 3 = 3.6e-6.
"""
import numpy as np
import pytest

import oracle
import parity_bars as bars
from paper_2105_08722_amd import encore

pytestmark = pytest.mark.gpu

N_POINTS, BOX = 300_000, 700.0


@pytest.fixture(scope="module")
def ctx():
    c = encore.Context(0)
    yield c
    c.close()


@pytest.fixture(scope="module")
def catalog():
    rng = np.random.default_rng(23)
    pos, w = rng.uniform(0.0, BOX, (N_POINTS, 3)), rng.uniform(0.5, 1.5, N_POINTS)
    return pos, w, rng.choice(N_POINTS, 24, replace=False)


@pytest.mark.parametrize("lmax,group", [(0, 4), (1, 4), (2, 6), (3, 5), (4, 3)])
def test_alm_wide_groups(ctx, catalog, lmax, group):
    pos, w, prim = catalog
    for nbins in (1, group - 1, group, group + 1, 2 * group + 1):
        print("[scattered] lmax %d nbins %d" % (lmax, nbins), flush=True)
        edges = np.linspace(6.0, 26.0, nbins + 1)
        ao = oracle.alm(pos, w, lmax, edges, box=BOX, primaries=prim)
        with encore.build_grid(ctx, pos, w, r_max=edges[-1], box=BOX) as g:
            ag = encore.debug_alm(ctx, g, lmax, edges, prim, "splitbf16")
        assert np.max(np.abs(ag - ao)) <= 3.6e-6 * np.max(np.abs(ao)), nbins


def test_same_bits_alone_batched_sliced(ctx, catalog, monkeypatch):
    pos, w, _ = catalog
    rng = np.random.default_rng(4)
    prim = rng.choice(N_POINTS, 700, replace=False)
    edges = np.linspace(6.0, 30.0, 9)
    N, lmax, prec = 4, 3, "splitbf16"
    print("[scattered] batch", flush=True)
    with encore.build_grid(ctx, pos, w, r_max=edges[-1], box=BOX) as g, \
            encore.build_grid(ctx, pos[:40_000], w[:40_000], r_max=edges[-1], box=BOX) as small:
        alone = encore.npcf(ctx, g, N, lmax, edges, precision=prec, primaries=prim)
        other = encore.npcf(ctx, small, N, lmax, edges, precision=prec)
        part = encore.npcf(ctx, small, N, lmax, edges, precision=prec, primaries=prim[prim < 40_000])
        z = encore.npcf_batch(ctx, [small, g, small, g], N, lmax, edges, precision=prec,
                              primaries=[None, prim, prim[prim < 40_000], prim])
        assert np.array_equal(z[0], other) and np.array_equal(z[1], alone)
        assert np.array_equal(z[2], part) and np.array_equal(z[3], alone)
        assert np.array_equal(encore.npcf(ctx, g, N, lmax, edges, precision=prec, primaries=prim, noalloc=True), alone)
        pairs = ctx.last_timings()["pairs"]
        monkeypatch.setenv("ENCORE_MAX_SLICE_ROWS", "256")
        assert np.array_equal(encore.npcf(ctx, g, N, lmax, edges, precision=prec, primaries=prim), alone)
        monkeypatch.delenv("ENCORE_MAX_SLICE_ROWS")
        for force in ("0", "1"):
            monkeypatch.setenv("ENCORE_GATHER_PERSISTENT", force)
            assert np.array_equal(encore.npcf(ctx, g, N, lmax, edges, precision=prec, primaries=prim), alone)
            assert ctx.last_timings()["pairs"] == pairs
    few = prim[:40]
    with encore.build_grid(ctx, pos, w, r_max=edges[-1], box=BOX) as g:
        zg = encore.npcf(ctx, g, N, lmax, edges, precision=prec, primaries=few)
    zo, za = oracle.zeta(pos, w, N, lmax, edges, box=BOX, primaries=few, return_abs=True)
    bars.check(zg, zo, za, prec, "scattered primaries")
