"""The gather over every shape of bin groups: bin counts that leave a ragged last
group, one group, and counts whose groups would repeat with the period of the shader
engines, at the degrees where the bins per work item or the split over m changes.

Tolerances, of the largest coefficient: FP64 1e-12 (rounding order).  FP32 terms with
FP64 sums 1e-6 (a term's own rounding, about 10 operations of 6e-8).  The plain FP32
sums of the split-bf16 path: at most 3000 / 64 + 6 additions per lane and lane tree,
each 6e-8 of a partial sum that is at most sqrt(2 lmax + 1) times the monopole's:
53 * 6e-8 * sqrt(19) = 1.4e-5.
"""
import numpy as np
import pytest

import oracle
import parity_bars as bars
from paper_2105_08722_amd import encore

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-6, "splitbf16": 1.4e-5}


@pytest.fixture(scope="module")
def ctx():
    c = encore.Context(0)
    yield c
    c.close()


def _catalog():
    rng = np.random.default_rng(41)
    return rng.uniform(0.0, 100.0, (3000, 3)), rng.uniform(0.5, 1.5, 3000)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "splitbf16"])
@pytest.mark.parametrize("lmax", [0, 1, 2, 4, 6, 7, 9])
def test_alm_over_bin_counts(ctx, lmax, precision):
    pos, w = _catalog()
    prim = np.arange(5, 3000, 171)
    for nbins in (1, 2, 3, 8, 13, 16):
        print("[groups] lmax %d nbins %d %s" % (lmax, nbins, precision), flush=True)
        edges = np.linspace(3.0, 28.0, nbins + 1)
        ao = oracle.alm(pos, w, lmax, edges, box=100.0, primaries=prim)
        with encore.build_grid(ctx, pos, w, r_max=edges[-1], box=100.0) as g:
            for full in (False, True):   # few primaries, and every point in one launch
                ag = encore.debug_alm(ctx, g, lmax, edges, prim, precision, full_launch=full)
                assert np.max(np.abs(ag - ao)) <= TOL[precision] * np.max(np.abs(ao)), (nbins, full)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "splitbf16"])
def test_accepted_pairs(ctx, precision):
    """The accepted-pair count is the number of pairs inside the bins, whatever the
    groups (a ragged group's missing bins hold none)."""
    pos, w = _catalog()
    pos, w = pos[:1500], w[:1500]
    d = pos[:, None] - pos[None]
    d -= 100.0 * np.round(d / 100.0)
    r2 = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]
    for nbins in (2, 3, 4, 7, 11):
        edges = np.linspace(3.0, 28.0, nbins + 1)
        want = int(((r2 >= edges[0] ** 2) & (r2 < edges[-1] ** 2)).sum())
        for lmax in (1, 4, 8):
            print("[groups] pairs nbins %d lmax %d %s" % (nbins, lmax, precision), flush=True)
            with encore.build_grid(ctx, pos, w, r_max=edges[-1], box=100.0) as g:
                encore.npcf(ctx, g, 3, lmax, edges, precision=precision)
            assert ctx.last_timings()["pairs"] == want, (nbins, lmax)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "splitbf16"])
@pytest.mark.parametrize("lmax", [0, 1, 3, 4, 5, 7, 10])
def test_persistent_grid_equals_static(ctx, monkeypatch, lmax, precision):
    """The grid of the gather (one wave per item, or resident waves pulling items)
    changes no bit of the result and no pair of the count, with one job and with
    several of uneven size; the result is the oracle's."""
    print("[groups] grids lmax %d %s" % (lmax, precision), flush=True)
    pos, w = _catalog()
    edges = np.linspace(3.0, 28.0, 6)
    got = []
    for force in ("0", "1"):
        monkeypatch.setenv("ENCORE_GATHER_PERSISTENT", force)
        grids = [encore.build_grid(ctx, pos[:k], w[:k], r_max=edges[-1], box=100.0) for k in (900, 31, 1500)]
        try:
            z = encore.npcf_batch(ctx, grids, 3, lmax, edges, precision=precision)
            pairs = ctx.last_timings()["pairs"]
            one = encore.npcf(ctx, grids[0], 3, lmax, edges, precision=precision)
        finally:
            for g in grids:
                g.free()
        assert np.array_equal(one, z[0])
        got.append((z, pairs))
    assert np.array_equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]
    zo, za = oracle.zeta(pos[:900], w[:900], 3, lmax, edges, box=100.0, return_abs=True)
    bars.check(got[0][0][0], zo, za, precision, "lmax %d" % lmax)
