"""What calls promise at the edges of their inputs, settings and budgets."""
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


# ---- batches whose second half does not fit the budget at first ---------------

def _jobs(cc, dims, npts, nbins, iters=2):
    specs = []
    for q, (d, n) in enumerate(zip(dims, npts)):
        a, u = W.genz_params(q % 5, d, 70 + q)
        specs.append(dict(method=0, ndim=d, family=q % 5, a=a, u=u, seed=q + 1, nstart=n,
                          maxeval=iters * n, nbins=nbins, flags=cc.FP64))
    return specs


@pytest.mark.parametrize("budget_mib", [12, 14, 16])
def test_batch_retried_after_one_half_is_queued(cc, ctx, budget_mib):
    # the first half is one integral (8 MiB of tile rows), whose setup launch is
    # queued when the second half's 11 MiB of rows are refused; the retry gives
    # that integral's buffers to other engines (1.4 MiB of rows for the second half)
    specs = _jobs(cc, [16] * 12, [700000] + [1 << 16] * 11, 256)
    want = cc.vegas_batch(ctx, specs)
    for _ in range(3):
        c = cc.Context(hbm_budget=budget_mib << 20)
        got = cc.vegas_batch(c, specs)
        c.close()
        for r, w in zip(got, want):
            assert r["status"] == 0 and r["neval"] == w["neval"] and r["fail"] == w["fail"]
            for k, tol in (("integral", 1e-12), ("error", 1e-11)):
                assert abs(r[k] - w[k]) <= tol * abs(w[k]), k


def test_state_file_of_more_iterations_is_refused(cc, ctx, tmp_path):
    # a call refused once its engine is set up leaves the context as it was
    a, u = W.genz_params(W.GAUSSIAN, 4, 1)
    path = str(tmp_path / "vegas.state")
    kw = dict(ctx=ctx, nbins=64, nstart=2000, seed=3)
    cc.vegas(W.GAUSSIAN, a, u, statefile=path, maxeval=12000, **kw)
    want = cc.vegas(W.GAUSSIAN, a, u, maxeval=6000, **kw)
    for _ in range(3):
        with pytest.raises(cc.CcubaError):
            cc.vegas(W.GAUSSIAN, a, u, statefile=path, maxeval=6000, **kw)
        specs = _jobs(cc, [4, 4], [2000, 2000], 64)
        again = cc.vegas_batch(ctx, specs)
        assert [r["status"] for r in again] == [0, 0]
        got = cc.vegas(W.GAUSSIAN, a, u, maxeval=6000, **kw)
        assert abs(got["integral"] - want["integral"]) <= 1e-12 * abs(want["integral"])


# ---- an integral's bits do not depend on the batch's other integrals ----------

def _run_fixed_point(cc, dims, npts, nbins):
    # tiles of 256 points whatever the batch, one engine, and the histogram whose
    # sums do not depend on the order of their adds: the values are all within
    # the window that its integers hold (v^2 down to 2^-37 of the cap), so that
    # none goes to the FP64 histogram beside it
    specs = _jobs(cc, dims, npts, nbins, iters=6)
    for s in specs:
        s["family"], s["a"] = W.C0, np.full(s["ndim"], 0.2)
    c = cc.Context()
    for key, value in (("min_tile", 256), ("hist64", 0), ("batch_streams", 1)):
        c.config(key, value)
    res = cc.vegas_batch(c, specs)
    c.close()
    return res


@pytest.mark.parametrize("nbins", [255, 256])
def test_fixed_point_histogram_beside_a_larger_integral(cc, nbins):
    # d = 16 with so many bins leaves no room for the fixed-point histogram; the
    # others, of the same number of Philox blocks, keep theirs
    dims, npts = [15, 14, 13, 16], [16384, 9999, 12000, 16000]
    few = _run_fixed_point(cc, dims[:3], npts[:3], nbins)
    many = _run_fixed_point(cc, dims, npts, nbins)
    for a, b in zip(few, many):
        assert a["status"] == b["status"] == 0
        assert a["integral"] == b["integral"] and a["error"] == b["error"]


@pytest.mark.parametrize("npts", [256, 8192, 8193, 16384])
def test_tile_sums_with_and_without_the_fold(cc, npts):
    # 1, 32, 33 and 64 tiles: summed by the refine launch alone, or through the fold
    # where another integral of the batch has more
    few = _run_fixed_point(cc, [3, 4, 2], [npts] * 3, 64)
    many = _run_fixed_point(cc, [3, 4, 2, 5], [npts] * 3 + [40000], 64)
    for a, b in zip(few, many):
        assert a["status"] == b["status"] == 0
        assert a["integral"] == b["integral"] and a["error"] == b["error"]


# ---- Suave: regions whose values leave the normal range ------------------------

@pytest.mark.parametrize("a,nsplit,flatness", [((36.0, 3.0), 64, 25.0), ((3.0, 36.0), 64, 25.0),
                                               ((35.7, 20.0), 64, 25.0),
                                               ((36.0, 1.0, 36.0), 8, 2.5)])
def test_suave_halves_of_subnormal_values(cc, ctx, a, nsplit, flatness):
    # a Gaussian's tail from e^-324 to e^-729: halves whose deviations from their
    # mean are subnormal, or all zero, beside others in the normal range
    d, u = len(a), np.zeros(len(a))
    kw = dict(seed=1, nnew=1000, nbins=32, nsplit=nsplit, flatness=flatness, maxeval=15000)
    g = cc.suave(W.GAUSSIAN, np.array(a), u, ctx=ctx, trace=True, **kw)
    o = O.suave(O.genz(W.GAUSSIAN, np.array(a), u), d, **kw)
    assert g["nregions"] == o["nregions"] and g["neval"] == o["neval"] and g["fail"] == o["fail"]
    assert np.array_equal(g["cut"], o["cut"]) and np.array_equal(g["lo"], o["lo"])
    assert abs(g["integral"] - o["integral"]) <= 1e-12 * abs(o["integral"])
    assert abs(g["error"] - o["error"]) <= 1e-10 * abs(o["error"])


# ---- a Cuhre store that grows under a tight budget ------------------------------

def test_cuhre_store_grows_beside_no_more_than_it_needs(cc, ctx):
    # 36600 KiB hold the old store and the new one, and then the new one's scratch,
    # but not all three at once
    a, u = W.genz_params(W.GAUSSIAN, 3, 3)
    kw = dict(epsrel=1e-30, maxeval=33 * 200000, max_regions_per_batch=20000)
    c = cc.Context(hbm_budget=36600 << 10)
    g = cc.cuhre(W.CORNER_PEAK, a, u, ctx=c, **kw)
    c.close()
    w = cc.cuhre(W.CORNER_PEAK, a, u, ctx=ctx, **kw)
    assert g["nregions"] == w["nregions"] and g["neval"] == w["neval"] and g["fail"] == w["fail"]
    assert abs(g["integral"] - w["integral"]) <= 1e-12 * abs(w["integral"])
    assert abs(g["error"] - w["error"]) <= 1e-10 * abs(w["error"])


# ---- a device integrand's arrays --------------------------------------------------

@pytest.mark.parametrize("nvec,npts", [(1000, 1000), (1000, 3500), (4096, 12288)])
def test_device_integrand_may_keep_its_first_arrays(cc, ctx, nvec, npts):
    # as one does that replays a graph recorded over them; a shorter last batch is
    # their first part.  It only multiplies, so that both sides compute the same bits
    kw = dict(ctx=ctx, nvec=nvec, nstart=npts, maxeval=4 * npts, nbins=64, seed=4)
    kept, sizes = [], []

    def fdev(x, f):
        if not kept:
            kept.extend((x, f))
        m = len(x)
        sizes.append(m)
        xk, fk = kept
        fk[:m, 0] = xk[:m, 0] * xk[:m, 1]

    g = cc.vegas_batched(fdev, 3, 1, where="device", **kw)
    h = cc.vegas_batched(lambda x: x[:, 0] * x[:, 1], 3, 1, **kw)
    assert max(sizes) == sizes[0] and g["neval"] == h["neval"] == 4 * npts
    assert abs(g["integral"] - h["integral"]) <= 1e-12 * abs(h["integral"])
    assert abs(g["error"] - h["error"]) <= 1e-10 * abs(h["error"])


# ---- device sources: the last trip of a tile ---------------------------------------

LOOP_SRC = r"""
__device__ double ccuba_user(const double *x, int d, const double *a, const double *u) {
  double s = 0.0;
  for (int j = 0; j < d; ++j) {
    const double t = x[j] - u[j];
    s = fma(a[j] * a[j], t * t, s);
  }
  return exp(-s);
}
"""


@pytest.mark.parametrize("d,nbins,npts,ilp", [
    (3, 64, 255, 2), (3, 64, 257, 2), (8, 128, 511, 2), (11, 128, 513, 2), (11, 100, 40961, 2),
    (16, 256, 2049, 2), (13, 64, 1025, 1)])
def test_source_with_points_left_over(cc, d, nbins, npts, ilp):
    # (the bars of the integrator's parity tests)
    a, u = W.genz_params(W.GAUSSIAN, d, 21)
    kw = dict(nbins=nbins, nstart=npts, maxeval=5 * npts, seed=9)
    c = cc.Context()
    c.config("ilp", ilp)
    s = cc.vegas_source(LOOP_SRC, d, a, u, ctx=c, **kw)
    b = cc.vegas(W.GAUSSIAN, a, u, ctx=c, **kw)
    c.close()
    assert s["neval"] == b["neval"] == 5 * npts and s["fail"] == b["fail"]
    for k, tol in (("integral", 1e-12), ("error", 1e-11)):
        assert abs(s[k] - b[k]) <= tol * abs(b[k]), k


@pytest.mark.parametrize("epsrel", [0.0, 2e-3])
def test_engines_that_are_not_kept_match_the_kept_one(cc, epsrel):
    # their iterations are queued one by one, a kept engine's as graphs
    a, u = W.genz_params(W.GAUSSIAN, 3, 21)
    kw = dict(nbins=64, nstart=5000, maxeval=60 * 5000, epsrel=epsrel, seed=9)
    c = cc.Context()
    kept = cc.vegas(W.GAUSSIAN, a, u, ctx=c, **kw)
    c.config("engine_cache", 0)
    runs = [cc.vegas(W.GAUSSIAN, a, u, ctx=c, **kw), cc.vegas_source(LOOP_SRC, 3, a, u, ctx=c, **kw)]
    c.close()
    for r in runs:
        assert r["neval"] == kept["neval"] and r["fail"] == kept["fail"]
        for k, tol in (("integral", 1e-12), ("error", 1e-11)):
            assert abs(r[k] - kept[k]) <= tol * abs(kept[k]), k


# ---- Cuhre's rule: every split, at the edges of the sizes that choose it ------------

@pytest.mark.parametrize("d", [3, 4, 8])
@pytest.mark.parametrize("nreg", [511, 512, 49151, 49152, 49217])
def test_oscillatory_rule_at_the_edges_of_its_splits(cc, ctx, d, nreg):
    # regions repeated in blocks of 61, so that the oracle evaluates 61 of them (the
    # bars of the rule's own parity test)
    rng = np.random.default_rng(d)
    a, u = W.genz_params(W.OSCILLATORY, d, 5)
    c0, h0 = rng.uniform(0.2, 0.8, (61, d)), rng.uniform(0.01, 0.2, (61, d))
    pick = np.arange(nreg) % 61
    g = cc.cuhre_rule(ctx, W.OSCILLATORY, a, u, c0[pick], h0[pick])
    for q in range(61):
        o = O.gm_rule(O.genz(W.OSCILLATORY, a, u), c0[q], h0[q])
        same = pick == q
        vol = np.prod(2.0 * h0[q])
        for k, m in (("I7", 20), ("I5", 60)):
            assert np.all(np.abs(g[k][same] - o[k]) <= 1e-12 * abs(o[k]) + 1e-15 * vol * m), k
        D = np.sort(o["dfour"])[::-1]
        if D[0] - D[1] > 1e-9 * D[0]:
            assert np.all(g["axis"][same] == o["axis"])


# ---- the sizes where a single integral's tiles change ---------------------------------

@pytest.mark.parametrize("d,nbins,npts", [(3, 64, 2 << 20), (3, 64, (2 << 20) + 1),
                                          (2, 64, 24576 * 256 + 1), (16, 256, 65537),
                                          (16, 256, 3072 * 256 + 1)])
def test_tiles_of_a_single_integral_at_its_edges(cc, ctx, d, nbins, npts):
    # one and two tiles per compute unit, the setting's three, and the one block that
    # a compute unit holds at d = 16 (the bars of the integrator's parity tests)
    a, u = W.genz_params(W.GAUSSIAN, d, 12)
    kw = dict(nbins=nbins, nstart=npts, maxeval=2 * npts, seed=6)
    g = cc.vegas(W.GAUSSIAN, a, u, ctx=ctx, **kw)
    o = O.vegas(O.genz(W.GAUSSIAN, a, u), d, **kw)
    assert g["neval"] == o["neval"] and g["fail"] == o["fail"]
    for k, tol in (("integral", 1e-12), ("error", 1e-11)):
        assert abs(g[k] - o[k]) <= tol * abs(o[k]), k


# ---- a served request holds what its launches read ------------------------------------

def test_served_request_in_a_small_budget(cc, ctx):
    # eight tile rows of 32 KiB, the grid, the history and the server's tables: 404 KiB,
    # and 32 KiB more with rows for a fold that a request of at most 64 tiles never has
    a, u = W.genz_params(W.GAUSSIAN, 16, 60)
    spec = dict(method=0, ndim=16, family=W.GAUSSIAN, a=a, u=u, seed=1, nstart=131072,
                maxeval=2 * 131072, nbins=256, flags=cc.FP64)
    c = cc.Context(hbm_budget=416 << 10)
    t = cc.submit(c, spec)
    cc.drain(c)
    r = cc.poll(c, t)
    c.close()
    w = cc.vegas_batch(ctx, [spec])[0]
    assert r["status"] == 0 and r["neval"] == w["neval"] and r["fail"] == w["fail"]
    for k, tol in (("integral", 1e-12), ("error", 1e-11)):
        assert abs(r[k] - w[k]) <= tol * abs(w[k]), k


# ---- profile mode: the rule's evaluations ----------------------------------------------

@pytest.mark.parametrize("fam,d,kw", [
    (W.GAUSSIAN, 2, dict(epsrel=1e-3, maxeval=10**6)),           # ends among the first states
    (W.GAUSSIAN, 3, dict(epsrel=1e-9, maxeval=10**6, max_regions_per_batch=100)),  # converges later
    (W.CORNER_PEAK, 3, dict(epsrel=1e-30, maxeval=33 * 20)),     # runs out of budget
    (W.GAUSSIAN, 10, dict(epsrel=1e-2, maxeval=10**6))])         # no shared first launch
def test_profiled_rule_evaluations_are_the_runs(cc, fam, d, kw):
    import bench
    a, u = W.genz_params(fam, d, 60 + d)
    c = cc.Context()
    c.config("profile", 1)
    bench._stats(cc, c)
    r = cc.cuhre(fam, a, u, ctx=c, **kw)
    st = bench._stats(cc, c)
    c.close()
    assert st.rule_evals == r["neval"] and st.rule_launches > 0 and st.rule_ms > 0.0


def test_batch_of_middle_sized_tiles_matches_the_integrals_alone(cc, ctx):
    # some 4 x 10^6 points an iteration at d N of about 2000: tiles between the
    # setting's smallest and a full one
    specs = _jobs(cc, [9, 10, 11, 12] * 8, [100003 + 1777 * q for q in range(32)], 200)
    for s, r in zip(specs, cc.vegas_batch(ctx, specs)):
        w = cc.vegas(s["family"], s["a"], s["u"], ctx=ctx, seed=s["seed"], nbins=200,
                     nstart=s["nstart"], maxeval=s["maxeval"])
        assert r["status"] == 0 and r["neval"] == w["neval"] and r["fail"] == w["fail"]
        for k, tol in (("integral", 1e-12), ("error", 1e-11)):
            assert abs(r[k] - w[k]) <= tol * abs(w[k]), k


# ---- Cuhre's selection: many candidates of one digit, and many tiles ---------------------

def _cuhre_as_the_oracle(cc, ctx, fam, d, regions, batch):
    a, u = W.genz_params(fam, d, 3)
    kw = dict(epsrel=1e-30, maxeval=(2**d + 2 * d * d + 2 * d + 1) * (2 * regions - 1),
              max_regions_per_batch=batch)
    g = cc.cuhre(fam, a, u, ctx=ctx, **kw)
    o = O.cuhre(O.genz(fam, a, u), d, **kw)
    assert g["nregions"] == o["nregions"] and g["neval"] == o["neval"] and g["fail"] == o["fail"]
    assert abs(g["integral"] - o["integral"]) <= 1e-12 * abs(o["integral"])
    assert abs(g["error"] - o["error"]) <= 1e-10 * o["error"] + 1e-14 * abs(o["integral"])


@pytest.mark.parametrize("fam,d,regions,batch", [(W.OSCILLATORY, 5, 60000, 9000),
                                                 (W.OSCILLATORY, 3, 200000, 30000),
                                                 (W.GAUSSIAN, 2, 300000, 90000),
                                                 (W.C0, 2, 300000, 90000)])
def test_cuhre_with_many_candidates_matches_oracle(cc, ctx, fam, d, regions, batch):
    # the errors of a smooth integrand share few digits: thousands of candidates for
    # the last places, beyond what the ranking holds in registers too
    _cuhre_as_the_oracle(cc, ctx, fam, d, regions, batch)


def test_cuhre_with_many_tiles_matches_oracle(cc, ctx):
    # the last step selects among 4.5 x 10^6 positions: 4392 tiles, counted by a launch of their own
    _cuhre_as_the_oracle(cc, ctx, W.OSCILLATORY, 2, 2848576, 1200000)
