"""The autotuner times its sample on the grid that a pass over every point launches:
the persistent one from 262,144 work items on, where that kernel exists."""
import numpy as np
import pytest

from paper_2105_08722_amd import encore

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,N,lmax,nbins,precision,persistent", [
    (140_000, 3, 2, 4, "fp64", True),     # 280,000 items of two bins
    (100_000, 3, 2, 4, "fp64", False),    # 200,000
    (140_000, 3, 5, 4, "fp64", False),    # no persistent kernel
])
def test_sample_takes_the_full_passes_grid(n, N, lmax, nbins, precision, persistent):
    print("[autotune-grid] n %d lmax %d %s" % (n, lmax, precision), flush=True)
    rng = np.random.default_rng(9)
    pos, w = rng.uniform(0.0, 400.0, (n, 3)), np.ones(n)
    edges = np.linspace(4.0, 20.0, nbins + 1)
    with encore.Context(0) as c:
        rep = encore.autotune(c, pos, w, N, lmax, edges, box=400.0, precision=precision, n_sample=2000)
        assert rep["persistent"] == persistent
        assert 0.0 < rep["best_ms"] <= rep["default_ms"]
        with encore.build_grid(c, pos, w, r_max=edges[-1], box=400.0) as g:
            assert np.all(np.isfinite(encore.npcf(c, g, N, lmax, edges, precision=precision, primaries=np.arange(50))))
