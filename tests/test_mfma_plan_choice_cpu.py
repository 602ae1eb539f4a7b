"""The 4PCF's split-BF16 plan takes one class per m of the last factor where classes by
the parity of its l would only pad more row tiles, and classes by parity where those
halve the output tiles: output tiles of the plan (with the padding of its wave jobs)."""
import pytest

from paper_2105_08722_amd import encore


@pytest.mark.parametrize("lmax,nbins,allp,tiles", [
    (2, 6, False, 13 * 4),      # by parity 20 wave jobs of 4 tiles
    (3, 6, False, 27 * 4),      # 34
    (4, 4, True, 31 * 4),       # 37
    (5, 10, False, 1660),       # one class per m 2008
    (4, 12, True, 2208),        # 344 + 241 + 113 + 10 wave jobs instead of 483 + 69
])
def test_plan_tiles(lmax, nbins, allp, tiles):
    assert encore.mfma_plan_stats(4, lmax, nbins, allp)["dense_entries"] == 256 * tiles
