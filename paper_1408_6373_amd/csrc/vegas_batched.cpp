// vegas_batched.cpp -- Vegas with a caller-evaluated integrand.
//
// The accelerator strategy of Sect. 3.2.4: the integrand receives batches of
// exactly nvec points, fewer only in an iteration's last batch, as
// x[nvec][ndim] with f[nvec][ncomp] to fill (the integrand declaration of
// Sect. 3.2.2, core < 0 for an accelerator).  The library makes each batch's
// points on the GPU with the points kernel (the Philox words, uniforms and
// grid map of DoSample) and hands them over in host memory or, for an
// integrand that runs its own GPU code, in device memory.  The rest of the
// iteration stays on the GPU: per-tile sums of every component and component
// 0's histogram, the fold kernel over those rows, and one workgroup for the
// statistics, the stop rule and the grid, which also writes the states to the
// pinned block.
//
// The integrand gets the same arrays for every batch, so that a program may keep
// their addresses (in a graph it replays, say); a batch's points are therefore
// made when the one before it has been evaluated, except that an iteration's first
// are queued behind the last one's statistics.  3 iterations of 4 batches of 10^6
// points at d = 8, a Gaussian in five library kernels: 2.02 ms, 1.39 ms of it the
// integrand's own; 1.92 ms with the next batch made meanwhile in a second set of
// arrays, which such a program would not see.
#include "vegas_batched.h"

#include <algorithm>

#include "noalloc.h"
#include "vegas.h"
#include "vegas_engine.h"

namespace ccuba {

namespace {

constexpr int kBatchedTile = 4096;  // points per tile row

// An iteration's first points are made before it is known that the last one was
// not enough, for batches up to this size.  Larger ones run long enough to hide
// the wait: 256 MiB are about 3.5 x 10^6 points at d = 8, whose kernels take
// 0.1 ms, the wait 0.01 ms.
constexpr long long kAheadBytes = 256ll << 20;

// Nothing of the call is left on the stream when its buffers go back.
struct Drain {
  hipStream_t s;
  ~Drain() { (void)hipStreamSynchronize(s); }
};

struct PinnedHost {
  void *p = nullptr;
  ~PinnedHost() {
    if (p) (void)hipHostFree(p);
  }
};

long long ceil_div(long long a, long long b) { return (a + b - 1) / b; }

}  // namespace

int vegas_batched(ccuba_ctx *ctx, const BatchedSpec &sp, ccuba_batch_integrand fn,
                  void *userdata, long long *neval, int *fail, double integral[],
                  double error[], double prob[]) {
  hipStream_t s = ctx->stream;
  const int d = sp.ndim, N = sp.nbins, nc = sp.ncomp, dN = d * N, R = 2 * nc + dN;
  const int row = N + 1;
  for (int c = 0; c < nc; ++c) integral[c] = error[c] = prob[c] = 0.0;
  VegasSpec vs;
  vs.nstart = sp.nstart;
  vs.nincrease = sp.nincrease;
  vs.maxeval = sp.maxeval;
  int iters = 0;
  long long nmax = 0;
  vegas_budget(vs, &iters, &nmax);
  if (iters == 0) {  // not even one iteration fits the budget
    *neval = 0;
    *fail = 1;
    return CCUBA_OK;
  }
  const int cap = iters;
  const long long mmax = std::min<long long>(sp.nvec, nmax);
  const long long tiles_max = ceil_div(nmax, sp.nvec) * ceil_div(mmax, kBatchedTile);
  const long long groups_max = ngroups_of((int)tiles_max);
  DevBuf<double> grid, x, f, w, rows, ghist, gsums, hist;
  // all zero: the components' states before the first iteration, and what the
  // fold's view of the tile rows reads, a state that is never done and tile
  // sums of zero
  DevBuf<double> zeros;
  DevBuf<VJob> view;
  DevBuf<long long> task_end;
  static_assert(sizeof(VState) % sizeof(double) == 0, "whole doubles");
  const long long stw = sizeof(VState) / sizeof(double);
  const long long nzero = (nc + 1) * stw + 2 * tiles_max;
  int rc;
  if ((rc = grid.alloc(ctx, (size_t)d * row)) || (rc = x.alloc(ctx, mmax * d)) ||
      (rc = f.alloc(ctx, mmax * nc)) || (rc = w.alloc(ctx, mmax)) ||
      (rc = rows.alloc(ctx, tiles_max * R)) || (rc = ghist.alloc(ctx, groups_max * R)) ||
      (rc = gsums.alloc(ctx, 2 * groups_max)) || (rc = hist.alloc(ctx, 2ll * nc * cap)) ||
      (rc = zeros.alloc(ctx, nzero)) || (rc = view.alloc(ctx, 1)) ||
      (rc = task_end.alloc(ctx, 1)))
    return rc;
  VState *const states = (VState *)zeros.p, *const dummy = states + nc;
  double *const tzero = zeros.p + (nc + 1) * stw;
  PinnedHost xh, fh;
  const bool host = sp.where == CCUBA_POINTS_HOST;
  if (host) {
    CCUBA_HIP(hipHostMalloc(&xh.p, mmax * d * sizeof(double), hipHostMallocDefault));
    CCUBA_HIP(hipHostMalloc(&fh.p, mmax * nc * sizeof(double), hipHostMallocDefault));
  }
  const bool ahead = mmax * (d + nc + 1) * (long long)sizeof(double) <= kAheadBytes;
  double *pin_host = nullptr, *pin_dev = nullptr;
  if ((rc = pinned_block(ctx, &pin_host, &pin_dev))) return rc;
  static_assert(kMaxComp * sizeof(VState) <= ccuba_ctx::kPinnedBytes, "the states fit");
  const VState *const out = (const VState *)pin_host;
  Drain drain{s};
  CCUBA_HIP(launch_init_grid(grid.p, d, N, s));
  CCUBA_HIP(hipMemsetAsync(zeros.p, 0, nzero * sizeof(double), s));

  PointsArgs pa{};
  pa.ndim = d;
  pa.nbins = N;
  pa.prec = sp.prec;
  pa.key0 = (uint32_t)(sp.seed & 0xffffffffull);
  pa.key1 = (uint32_t)(sp.seed >> 32);
  pa.sid = sp.sid;
  pa.grid = grid.p;
  pa.x = x.p;
  pa.w = w.p;
  // the points of the batch of iteration t (of n points) that starts at i0
  auto make_points = [&](int t, long long n, long long i0) {
    pa.iteration = t;
    pa.i0 = i0;
    pa.npts = std::min<long long>(sp.nvec, n - i0);
    return launch_points(pa, s);
  };
  VJob jv{};
  long long tend = 0;
  long long handed = 0;  // points given to the integrand
  const int core = -1;   // an accelerator (Sect. 3.2.4)
  bool made = true;   // the next batch's points are launched
  bool ready = false; // and there
  CCUBA_HIP(make_points(0, sp.nstart, 0));
  for (int t = 0; t < iters; ++t) {
    const long long n = sp.nstart + (long long)t * sp.nincrease;
    int tiles = 0;
    for (long long i0 = 0; i0 < n; i0 += sp.nvec) {
      const long long m = std::min<long long>(sp.nvec, n - i0);
      if (!made) CCUBA_HIP(make_points(t, n, i0));
      if (host)
        CCUBA_HIP(hipMemcpyAsync(xh.p, x.p, m * d * sizeof(double), hipMemcpyDeviceToHost, s));
      // (the last batch's values, which f holds, have been read then, too)
      if (host || !ready) CCUBA_HIP(hipStreamSynchronize(s));
      made = ready = false;
      const int mi = (int)m, nd = d, ncomp = nc;
      const int urc = host ? fn(&nd, (const double *)xh.p, &ncomp, (double *)fh.p, userdata, &mi,
                                &core)
                           : fn(&nd, x.p, &ncomp, f.p, userdata, &mi, &core);
      handed += m;
      if (urc == -999) {
        for (int c = 0; c < nc; ++c) integral[c] = error[c] = prob[c] = 0.0;
        *neval = handed;
        *fail = -99;
        return CCUBA_OK;
      }
      if (host)
        CCUBA_HIP(hipMemcpyAsync(f.p, fh.p, m * nc * sizeof(double), hipMemcpyHostToDevice, s));
      BatchedArgs ba{d, N, nc, sp.prec, m, kBatchedTile, tiles, w.p, f.p,
                     pa.key0, pa.key1, pa.sid, t, i0, rows.p, states};
      CCUBA_HIP(launch_batched_accumulate(ba, s));
      tiles += (int)ceil_div(m, kBatchedTile);
    }
    // the fold kernel sums the tile rows 32 at a time, seeing them as the
    // histogram rows of one job of R = 2 ncomp + ndim nbins bins
    const int ng = ngroups_of(tiles);
    if (tiles != jv.ntiles) {
      jv.ndim = 1;
      jv.nbins = R;
      jv.ntiles = tiles;
      jv.state = dummy;
      jv.thist = rows.p;
      jv.tsums = tzero;
      jv.ghist = ghist.p;
      jv.gsums = gsums.p;
      tend = (long long)ng * ((R + 63) / 64);
      JobSetup js{};
      js.job = jv;
      js.end = tend;
      js.job_dst = view.p;
      js.st_dst = dummy;
      js.end_dst = task_end.p;
      CCUBA_HIP(launch_job_setup(js, s));
    }
    FoldArgs fo{view.p, task_end.p, 1, tend, 0, nullptr, nullptr};
    CCUBA_HIP(launch_fold(fo, s));
    BatchedFinishArgs fa{};
    fa.ndim = d;
    fa.nbins = N;
    fa.ncomp = nc;
    fa.flags = sp.flags;
    fa.ngroups = ng;
    fa.ghist = ghist.p;
    fa.grid = grid.p;
    fa.state = states;
    fa.iter_I = hist.p;
    fa.iter_var = hist.p + (size_t)nc * cap;
    fa.hist_cap = cap;
    fa.nstart = sp.nstart;
    fa.nincrease = sp.nincrease;
    fa.mineval = sp.mineval;
    fa.maxeval = sp.maxeval;
    fa.epsrel = sp.epsrel;
    fa.epsabs = sp.epsabs;
    fa.out = (VState *)pin_dev;
    CCUBA_HIP(launch_batched_finish(fa, s));
    // the next iteration's first points, on the grid as refined
    made = ahead && t + 1 < iters;
    if (made) CCUBA_HIP(make_points(t + 1, n + sp.nincrease, 0));
    CCUBA_HIP(hipStreamSynchronize(s));
    ready = made;
    if (out[0].done) break;
  }
  for (int c = 0; c < nc; ++c) {
    integral[c] = out[c].integral;
    error[c] = out[c].error;
    prob[c] = out[c].prob;
  }
  *neval = out[0].neval;
  *fail = out[0].fail;
  return CCUBA_OK;
}

}  // namespace ccuba
