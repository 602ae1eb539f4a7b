"""The accepted-pair count where the gather runs as two launches, one per half of the
m range (lmax 9 and 10 with FP64 sums): each pair counts once."""
import numpy as np
import pytest

from paper_2105_08722_amd import encore

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32", "splitbf16"])
@pytest.mark.parametrize("lmax", [8, 9, 10])
def test_pairs_counted_once(lmax, precision):
    print("[pairs] lmax %d %s" % (lmax, precision), flush=True)
    rng = np.random.default_rng(17)
    pos, w = rng.uniform(0.0, 100.0, (700, 3)), rng.uniform(0.5, 1.5, 700)
    edges = np.linspace(3.0, 28.0, 4)
    d = pos[:, None] - pos[None]
    d -= 100.0 * np.round(d / 100.0)
    r2 = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]
    want = int(((r2 >= edges[0] ** 2) & (r2 < edges[-1] ** 2)).sum())
    with encore.Context(0) as ctx, encore.build_grid(ctx, pos, w, r_max=edges[-1], box=100.0) as g:
        encore.npcf(ctx, g, 3, lmax, edges, precision=precision)
        assert ctx.last_timings()["pairs"] == want
