"""What calls promise at the edges of their inputs, settings and budgets."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cc():
    import paper_1408_6373_amd as cc
    return cc


@pytest.fixture(scope="module")
def ctx(cc):
    c = cc.Context()
    yield c
    c.close()


# ---- refinement of rows without a usable sum ---------------------------------

@pytest.mark.parametrize("nbins", [2, 5, 64, 65, 256])
def test_refine_keeps_the_edges_of_rows_without_a_sum(cc, ctx, nbins):
    # a sum that is zero, negative or NaN keeps the edges, as in the oracle; an
    # infinite or overflowing one, whose shares place no edge, keeps them too
    rng = np.random.default_rng(nbins)
    H = rng.random((9, nbins)) + 0.1
    H[1, nbins // 2] = np.nan
    H[2] = np.nan
    H[3] = 0.0
    H[4, 0] = -2.0 * nbins
    H[5] = -1.0
    H[6, nbins - 1] = np.inf
    H[7] = 1.5e308
    grid = np.tile(np.linspace(0.0, 1.0, nbins + 1) ** 1.3, (9, 1))
    got = cc.vegas_refine(ctx, H, grid)
    for j in (1, 2, 3, 4, 5):
        assert np.array_equal(O.refine_dim(H[j], grid[j]), grid[j])
    for j in range(1, 8):
        assert np.array_equal(got[j], grid[j]), j
    for j in (0, 8):
        np.testing.assert_allclose(got[j], O.refine_dim(H[j], grid[j]), rtol=0, atol=1e-12)
