"""GPU kernels at the sizes where their splits and selections change, against
the oracle.  Tolerances are those of the integrator's own parity tests."""
import numpy as np
import pytest

import oracle as O
import workloads as W

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


@pytest.mark.parametrize("d,maxregions,nsplit", [(1, 40, 3), (3, 700, 150), (8, 330, 65),
                                                 (9, 70, 64), (3, 9000, 1024)])
def test_partition_ties_and_group_sizes(cc, ctx, d, maxregions, nsplit):
    # equal dyadic coefficients make spreads equal bit for bit in whole groups
    # of regions, so ties (lower position first) decide the selection; d = 8
    # and 9 are the last and first of the two search group sizes, and 9000
    # regions more than the selection holds in registers
    a, u = np.full(d, 0.5), np.zeros(d)
    kw = dict(seed=2, nsearch=16, niter=40, maxregions=maxregions, nsplit=nsplit)
    g = cc.divonne_partition(W.CORNER_PEAK, a, u, ctx=ctx, trace=True, **kw)
    o = O.divonne_partition(O.genz(W.CORNER_PEAK, a, u), d, **kw)
    assert g["nregions"] == o["nregions"] == maxregions and g["neval"] == o["neval"]
    assert np.array_equal(g["cut"], o["cut"])
    for k in ("lo", "hi", "xmin", "xmax"):
        assert np.array_equal(g[k], o[k]), k
    for k in ("fmin", "fmax", "spread"):
        assert np.allclose(g[k], o[k], rtol=1e-12, atol=0), k
