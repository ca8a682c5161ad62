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


def _suave_both(cc, ctx, fam, d, **kw):
    a, u = W.genz_params(fam, d, d + 40)
    g = cc.suave(fam, a, u, ctx=ctx, trace=True, **kw)
    o = O.suave(O.genz(fam, a, u), d, **kw)
    assert g["nregions"] == o["nregions"] and g["neval"] == o["neval"] and g["fail"] == o["fail"]
    assert np.array_equal(g["cut"], o["cut"]) and np.array_equal(g["lo"], o["lo"])
    for k, tol in (("integral", 1e-12), ("error", 1e-10)):
        assert abs(g[k] - o[k]) <= tol * abs(o[k]), k
    assert np.allclose(g["grid"], o["grid"], rtol=0, atol=1e-12)
    assert abs(g["prob"] - o["prob"]) < 1e-9


@pytest.mark.parametrize("d,nbins,nnew,nsplit,flatness", [
    (4, 64, 1023, 3, 25.0),     # one tile, a ragged chunk
    (5, 100, 1025, 1, 3.0),     # one more than the smallest piece
    (8, 256, 12289, 7, 50.0),   # several pieces, d = 4 nb
    (9, 128, 5000, 5, 2.5),     # the third dimension group, a fractional power
    (16, 256, 2500, 2, 64.0),   # LDS beyond the default limit
    (1, 3, 300000, 2, 1.0)])    # the most chunks, one dimension
def test_suave_pieces_match_oracle(cc, ctx, d, nbins, nnew, nsplit, flatness):
    _suave_both(cc, ctx, W.C0 if d % 2 else W.PRODUCT_PEAK, d, seed=d, nnew=nnew, nbins=nbins,
                nsplit=nsplit, flatness=flatness, maxeval=11 * nnew)


def test_suave_converging_run_matches_oracle(cc, ctx):
    # the run ends on its accuracy while the next step's statistics are queued
    _suave_both(cc, ctx, W.PRODUCT_PEAK, 3, seed=3, nnew=2000, nbins=32, nsplit=4, flatness=5.0,
                epsrel=2e-3, maxeval=10**6)


@pytest.mark.parametrize("fam,d,kw", [
    (W.GAUSSIAN, 2, dict(epsrel=1e-3, maxeval=10**6)),            # ends among the first states
    (W.CORNER_PEAK, 3, dict(epsrel=1e-30, maxeval=33 * 20)),      # the budget ends them
    (W.C0, 4, dict(epsrel=1e-30, maxeval=57 * 300, max_regions_per_batch=64)),  # the batch does
    (W.PRODUCT_PEAK, 5, dict(epsrel=1e-6, maxeval=10**6, max_regions_per_batch=2)),
    (W.OSCILLATORY, 10, dict(epsrel=1e-30, maxeval=1245 * 63)),   # corners beyond a wavefront
    (W.GAUSSIAN, 13, dict(epsrel=1e-30, maxeval=8557 * 7)),       # one doubling
    (W.C0, 15, dict(epsrel=1e-30, maxeval=33249 * 5)),            # no shared first launch
    (W.GAUSSIAN, 3, dict(epsrel=1e-3, mineval=33 * 40, maxeval=10**6))])
def test_cuhre_first_states_match_oracle(cc, ctx, fam, d, kw):
    a, u = W.genz_params(fam, d, 60 + d)
    g = cc.cuhre(fam, a, u, ctx=ctx, **kw)
    o = O.cuhre(O.genz(fam, a, u), d, **kw)
    assert g["nregions"] == o["nregions"] and g["neval"] == o["neval"] and g["fail"] == o["fail"]
    assert abs(g["integral"] - o["integral"]) <= 1e-12 * abs(o["integral"])
    assert abs(g["error"] - o["error"]) <= 1e-10 * o["error"] + 1e-14 * abs(o["integral"])


@pytest.mark.parametrize("d,a0,batch,regions", [(2, 30.0, 100, 900), (3, 40.0, 600, 1500),
                                                (3, 60.0, 1500, 3000), (2, 0.0, 100, 400)])
def test_cuhre_selection_of_tiny_errors_matches_oracle(cc, ctx, d, a0, batch, regions):
    # a narrow peak: errors from 1e-3 of their sum down past 2^-255 of it and to
    # exact zeros, with the boundary of the selection among the smallest (and,
    # for a constant, every error equal)
    a, u = np.full(d, a0), np.full(d, 0.3)
    npt = 2**d + 2 * d * d + 2 * d + 1
    kw = dict(epsrel=1e-30, mineval=npt * regions, maxeval=npt * regions,
              max_regions_per_batch=batch)
    g = cc.cuhre(W.GAUSSIAN, a, u, ctx=ctx, **kw)
    o = O.cuhre(O.genz(W.GAUSSIAN, a, u), d, **kw)
    assert g["nregions"] == o["nregions"] and g["neval"] == o["neval"] and g["fail"] == o["fail"]
    assert abs(g["integral"] - o["integral"]) <= 1e-12 * abs(o["integral"])
    assert abs(g["error"] - o["error"]) <= 1e-10 * o["error"] + 1e-14 * abs(o["integral"])


# ---- a device integrand's batches, the next one made ahead ------------------

@pytest.mark.parametrize("nbins,prec,nvec,nstart", [
    (64, 64, 1000, 1000),    # one batch an iteration
    (100, 64, 1000, 2001),   # the last batch one point; bins not a power of two
    (100, 32, 4096, 12288),  # whole batches of whole tiles, odd number of them
    (128, 32, 4097, 9000),   # ragged tiles
])
def test_device_batches_match_host_batches(cc, ctx, nbins, prec, nvec, nstart):
    # the integrand only multiplies, so that both sides compute the same bits,
    # and the sums differ only by the LDS histogram's order
    import torch
    flags = cc.FP32_EVAL if prec == 32 else cc.FP64
    kw = dict(ctx=ctx, nvec=nvec, nstart=nstart, nincrease=nvec, maxeval=5 * nstart + 10 * nvec,
              nbins=nbins, flags=flags, seed=4)
    seen = []

    def fdev(x, f):
        seen.append(len(x))
        f.copy_(torch.stack((x[:, 0] * x[:, 1], x[:, 2] * 0.5 + 0.25), 1))

    host = []

    def fhost(x):
        host.append(len(x))
        return np.stack((x[:, 0] * x[:, 1], x[:, 2] * 0.5 + 0.25), 1)

    g = cc.vegas_batched(fdev, 3, 2, where="device", **kw)
    h = cc.vegas_batched(fhost, 3, 2, **kw)
    assert seen == host and g["neval"] == h["neval"] and g["fail"] == h["fail"] == 1
    np.testing.assert_allclose(g["integral"], h["integral"], rtol=1e-12)
    np.testing.assert_allclose(g["error"], h["error"], rtol=1e-10)
    # an integrand that stops while the next batch's points are being made
    seen.clear()
    full = fdev

    def stop(x, f):
        full(x, f)
        return -999 if len(seen) == 2 else 0

    r = cc.vegas_batched(stop, 3, 2, where="device", **kw)
    assert r["fail"] == -99 and r["neval"] == sum(host[:2])
    again = cc.vegas_batched(fdev, 3, 2, where="device", **kw)
    np.testing.assert_allclose(again["integral"], h["integral"], rtol=1e-12)


# ---- DoSample: every dimension, both LDS layouts, what is left of a tile ----

def _rel(a, b):
    return abs(a - b) / max(abs(b), 1e-300)


def _all_dims(flags, nbins):
    specs = []
    for d in range(1, 17):
        a, u = W.genz_params(d % 5, d, 40 + d)
        n = 40961 + 127 * d
        specs.append(dict(method=0, ndim=d, family=d % 5, a=a, u=u, seed=d, nstart=n,
                          maxeval=3 * n, nbins=nbins, flags=flags))
    return specs


def _run_batch(cc, specs, ilp, hist64):
    c = cc.Context()
    c.config("ilp", ilp)
    c.config("hist64", hist64)
    res = cc.vegas_batch(c, specs)
    c.close()
    return res


@pytest.mark.parametrize("nbins,ilp,hist64", [
    (64, 2, 0),   # a fixed-point histogram of two words after the cells
    (256, 2, 0),
    (64, 1, 1),   # an FP64 histogram in its region before the cells
    (256, 1, 1),
    (2, 1, 0),
    (100, 2, 0),  # bins not a power of two: cells first
])
def test_every_dimension_in_one_batch(cc, nbins, ilp, hist64):
    # d = 1 to 16 with points that leave odd parts of trips and tiles; integrals of
    # all dimensions of a block count share a launch
    specs = _all_dims(cc.FP64, nbins)
    for s, r in zip(specs, _run_batch(cc, specs, ilp, hist64)):
        o = O.vegas(O.genz(s["family"], s["a"], s["u"]), s["ndim"], seed=s["seed"],
                    nstart=s["nstart"], maxeval=s["maxeval"], nbins=nbins)
        assert r["status"] == 0 and r["neval"] == o["neval"] and r["fail"] == o["fail"]
        assert _rel(r["integral"], o["integral"]) < 1e-12, s["ndim"]
        assert _rel(r["error"], o["error"]) < 1e-11, s["ndim"]


@pytest.mark.parametrize("nbins", [2, 64, 100, 256])
def test_fp32_layouts_and_trips_agree(cc, nbins):
    # FP32 evaluation: the points and their values are the same whatever the
    # histogram's type and place and the points per trip; only the order of the sums
    # differs (the bar of the fixed-point histogram's own test)
    specs = _all_dims(cc.FP32_EVAL, nbins)
    base = _run_batch(cc, specs, 1, 1)
    for ilp, hist64 in ((1, 0), (2, 0), (2, 1)):
        for s, r, b in zip(specs, _run_batch(cc, specs, ilp, hist64), base):
            assert r["status"] == 0 and r["neval"] == b["neval"] and r["fail"] == b["fail"]
            assert _rel(r["integral"], b["integral"]) < 1e-12, (ilp, hist64, s["ndim"])
            assert _rel(r["error"], b["error"]) < 1e-12, (ilp, hist64, s["ndim"])


@pytest.mark.parametrize("n", [65536, 65537, 3072 * 256, 3072 * 256 + 1])
def test_tiles_of_a_single_integral(cc, ctx, n):
    # the sizes where the tiles of an iteration change: 64 tiles and no fold up to
    # 65536 points, then one and two tiles per compute unit
    a, u = W.genz_params(0, 3, 12)
    kw = dict(nbins=64, nstart=n, maxeval=2 * n, seed=6)
    g = cc.vegas(0, a, u, ctx=ctx, **kw)
    o = O.vegas(O.genz(0, a, u), 3, **kw)
    assert g["neval"] == o["neval"] and g["fail"] == o["fail"]
    assert _rel(g["integral"], o["integral"]) < 1e-12
    assert _rel(g["error"], o["error"]) < 1e-11


# ---- memory budgets that refuse the rows of the smallest tiles --------------

def _wide(cc, n, jobs):
    # d = 16 with 256 bins: 32 KiB a tile row
    specs = []
    for q in range(jobs):
        a, u = W.genz_params(0, 16, 60 + q)
        specs.append(dict(method=0, ndim=16, family=0, a=a, u=u, seed=q + 1, nstart=n,
                          maxeval=2 * n, nbins=256, flags=cc.FP64))
    return specs


def test_batch_under_a_tight_budget_takes_larger_tiles(cc, ctx):
    # 8 x 65536 points: 8 MiB of rows of about 2048 points, 1 MiB of 16384
    specs = _wide(cc, 65536, 8)
    c = cc.Context(hbm_budget=6 << 20)
    before = c.config_get("min_tile")
    got = cc.vegas_batch(c, specs)
    assert c.config_get("min_tile") == before
    c.close()
    for r, w in zip(got, cc.vegas_batch(ctx, specs)):
        assert r["status"] == 0 and r["neval"] == w["neval"] and r["fail"] == w["fail"]
        assert _rel(r["integral"], w["integral"]) < 1e-12
        assert _rel(r["error"], w["error"]) < 1e-11


def test_served_request_under_a_tight_budget_takes_larger_tiles(cc, ctx):
    # 131072 points: 2 MiB in rows of 2048 points, 256 KiB of 16384
    spec = _wide(cc, 131072, 1)[0]
    c = cc.Context(hbm_budget=1536 << 10)
    t = cc.submit(c, spec)
    cc.drain(c)
    r = cc.poll(c, t)
    c.close()
    w = cc.vegas_batch(ctx, [spec])[0]
    assert r["status"] == 0 and r["neval"] == w["neval"] and r["fail"] == w["fail"]
    assert _rel(r["integral"], w["integral"]) < 1e-12
    assert _rel(r["error"], w["error"]) < 1e-11
