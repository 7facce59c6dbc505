"""Maxima and segmentation at the edges of their tiles (-m gpu): grids smaller than a tile,
tiles cut short to one cell along an axis, and fields of few distinct values, so
that the order of equal values (larger index first, also across the periodic
box's ends) decides most parents."""
import numpy as np
import pytest
import torch

from oracle import cwthf as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels", [3, 1000])
@pytest.mark.parametrize("n", [8, 9, 16, 17, 18, 32, 33, 34, 47, 49, 64, 65])
def test_tied_fields(n, levels):
    import paper_2501_10622_amd as hfm
    rng = np.random.default_rng(100 * n + levels)
    c = (rng.integers(0, levels, (n, n, n)) - levels // 2).astype(np.float32)
    c[c == 0] = np.where(rng.random(int((c == 0).sum())) < 0.5, 0.0, -0.0)  # equal to each other
    for tau in (0.0, -0.5):
        field = torch.as_tensor(c, device="cuda:0")
        assert np.array_equal(hfm.segment(field, tau).cpu().numpy(), O.segment(c, tau))
        assert np.array_equal(hfm.maxima(field, tau).cpu().numpy(), O.maxima(c, tau))
