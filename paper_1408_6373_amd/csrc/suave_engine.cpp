// suave_engine.cpp -- host driver of Suave (Sect. 3.2.2 prototype; the steps
// are those listed in suave.hip).
//
// Device memory: per region its bounds, grid and result, plus the nnew values
// and side bits of its own sample (10 bytes a point); the region count is
// bounded by the budget, R <= 1 + (maxeval - nnew) / (2 nnew).  A step's size
// follows from the budget alone, K = min(nsplit, R, (maxeval - neval) / (2
// nnew)); only the end of the run depends on the totals.  The part of a step
// that changes no region (selection and split statistics) is queued before
// the host has learned that the run goes on, so the device does not idle
// while the outcome travels.
#include "suave_engine.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "vegas_engine.h"

namespace ccuba {

int validate_suave(const SuaveSpec &s) {
  if (s.ndim < 1 || s.ndim > kMaxDim || s.nbins < 2 || s.nbins > kMaxBins || s.family < 0 ||
      s.family > C0 || s.nnew < 2 || s.nnew >= (1ll << 32) || !(s.flatness > 0.0) ||
      !std::isfinite(s.flatness) || s.nsplit < 1 || s.nsplit > kSuaveMaxSplit || s.mineval < 0 ||
      s.maxeval < 0 || !(s.epsrel >= 0.0) || !(s.epsabs >= 0.0))
    return CCUBA_EINVAL;
  for (int j = 0; j < s.ndim; ++j)
    if (!std::isfinite(s.a[j]) || !std::isfinite(s.u[j])) return CCUBA_EINVAL;
  return CCUBA_OK;
}

namespace {

// Points of a sampling tile and of a statistics chunk for a launch over `n'
// points of each of `regions' regions: about `groups' workgroups in all (what
// the device holds at once), so that a large launch runs in one round and a
// small one spreads, and at least `least' points, below which a workgroup's
// own setup and its row of results cost more than its points.
struct Pieces {
  int size, count;
};
Pieces pieces(long long n, long long regions, long long least, long long most, long long groups,
              long long multiple) {
  auto up = [&](long long v, long long m) { return (v + m - 1) / m * m; };
  const long long want = up((regions * n + groups - 1) / groups, multiple);
  const long long size = std::min(std::max(want, least), std::max(most, least));
  const long long count = (n + size - 1) / size;
  const long long even = up((n + count - 1) / count, multiple);
  return {(int)even, (int)((n + even - 1) / even)};
}

constexpr long long kTileMost = 1 << 20, kChunkMost = 8192, kChunkCount = 256;
// Sampling workgroups: as many as their LDS lets a compute unit hold, 4 at most
// (what their registers allow at d = 8).
Pieces tile_pieces(long long n, long long nchild, bool fine, int ncu, size_t lds) {
  const long long per_cu = std::max<long long>(1, std::min<long long>(4, 160 * 1024 / lds));
  return pieces(n, nchild, fine ? 1024 : 4096, kTileMost, per_cu * ncu, kSuaveBlock);
}
// (the chunks' partial sums are summed again by every workgroup: 256 at most)
Pieces chunk_pieces(long long n, long long K, bool fine, int ncu) {
  const long long least = std::max(fine ? 1024ll : 4096ll, (n + kChunkCount - 1) / kChunkCount);
  return pieces(n, K, least, kChunkMost, 4ll * ncu, 512);
}

struct Buffers {
  DevBuf<double> lo, hi, grid, I, var, chi2, inh_I, inh_var, v, fl1, fl2, hs, tsum, thist, p64;
  DevBuf<int> dof, sel, chpos, chser, cut;
  DevBuf<uint16_t> side;
};

}  // namespace

int run_suave(ccuba_ctx *ctx, const SuaveSpec &sp, SuaveResult &res, const SuaveTraceOut *tr,
              hipStream_t s) {
  int rc = validate_suave(sp);
  if (rc) return rc;
  res = SuaveResult();
  if (sp.nnew > sp.maxeval) return CCUBA_OK;  // no point can be afforded: fail 1
  const int d = sp.ndim, N = sp.nbins;
  const long long n = sp.nnew;
  const long long Rmax = 1 + (sp.maxeval - n) / (2 * n);
  if (Rmax > (1ll << 23)) return CCUBA_EINVAL;  // sampling serials are 24 bits
  const int Kmax = (int)std::min<long long>(sp.nsplit, std::max<long long>(1, Rmax - 1));
  const size_t dN = (size_t)d * N, row = (size_t)d * (N + 1);
  Buffers B;
  if ((rc = B.lo.alloc(ctx, Rmax * d)) || (rc = B.hi.alloc(ctx, Rmax * d)) ||
      (rc = B.grid.alloc(ctx, Rmax * row)) || (rc = B.I.alloc(ctx, Rmax)) ||
      (rc = B.var.alloc(ctx, Rmax)) || (rc = B.chi2.alloc(ctx, Rmax)) ||
      (rc = B.inh_I.alloc(ctx, Rmax)) || (rc = B.inh_var.alloc(ctx, Rmax)) ||
      (rc = B.dof.alloc(ctx, Rmax)) || (rc = B.v.alloc(ctx, Rmax * n)) ||
      (rc = B.side.alloc(ctx, Rmax * n)) || (rc = B.hs.alloc(ctx, (size_t)Kmax * d * 10)) ||
      (rc = B.p64.alloc(ctx, 2 * kParamRow)) || (rc = B.sel.alloc(ctx, Kmax)) ||
      (rc = B.chpos.alloc(ctx, 2 * Kmax)) || (rc = B.chser.alloc(ctx, 2 * Kmax)) ||
      (rc = B.cut.alloc(ctx, std::max<long long>(1, Rmax - 1))))
    return rc;
  // rows of partial results for the step of most of them; where the budget
  // refuses, larger pieces and fewer rows
  const size_t lds = suave_sample_lds(d, N) + 1024;
  bool fine = true;
  for (;; fine = false) {
    size_t trows = 0, crows = 0;
    for (long long k = 1; k <= Kmax; ++k) {
      trows = std::max<size_t>(trows, 2 * k * tile_pieces(n, 2 * k, fine, ctx->ncu, lds).count);
      crows = std::max<size_t>(crows, k * chunk_pieces(n, k, fine, ctx->ncu).count);
    }
    trows = std::max<size_t>(trows, tile_pieces(n, 1, fine, ctx->ncu, lds).count);  // the root
    if (!(rc = B.fl1.alloc(ctx, crows * d * 9)) && !(rc = B.fl2.alloc(ctx, crows * d * 2)) &&
        !(rc = B.tsum.alloc(ctx, trows * 2)) && !(rc = B.thist.alloc(ctx, trows * dN)))
      break;
    if (rc != CCUBA_ENOMEM || !fine) return rc;
    B.fl1.release();
    B.fl2.release();
    B.tsum.release();
    B.thist.release();
  }
  double *pin_host = nullptr, *pin_dev = nullptr;  // the totals land in host memory
  if ((rc = pinned_block(ctx, &pin_host, &pin_dev))) return rc;

  VegasSpec vs;
  vs.ndim = d;
  vs.family = sp.family;
  for (int j = 0; j < d; ++j) {
    vs.a[j] = sp.a[j];
    vs.u[j] = sp.u[j];
  }
  double p64[2][kParamRow];
  float p32[2][kParamRow];
  genz_constants(vs, p64, p32);
  CCUBA_HIP(hipMemcpyAsync(B.p64.p, p64, sizeof(p64), hipMemcpyHostToDevice, s));

  SuaveArgs A{};
  A.R = SRegions{B.lo.p, B.hi.p, B.grid.p, B.I.p, B.var.p, B.chi2.p, B.dof.p,
                 B.inh_I.p, B.inh_var.p, B.v.p, B.side.p};
  A.d = d;
  A.N = N;
  A.family = sp.family;
  A.flags = sp.flags & FLAG_FREEZE_GRID;
  A.nnew = n;
  A.key0 = (uint32_t)(sp.seed & 0xffffffffull);
  A.key1 = (uint32_t)(sp.seed >> 32);
  A.sid = sp.sid;
  A.flatness = sp.flatness;
  A.ipow = (sp.flatness == std::floor(sp.flatness) && sp.flatness <= 4096.0) ? (int)sp.flatness : 0;
  A.p64 = B.p64.p;
  A.sel = B.sel.p;
  A.chpos = B.chpos.p;
  A.chser = B.chser.p;
  A.fl1 = B.fl1.p;
  A.fl2 = B.fl2.p;
  A.hs = B.hs.p;
  A.tsum = B.tsum.p;
  A.thist = B.thist.p;
  A.cut = B.cut.p;
  // state t's totals and outcome go to slot t % 2 of the pinned block
  static_assert(sizeof(SState) <= 6 * sizeof(double), "a slot's totals");
  constexpr int kSlot = 8, kWord = 6;  // doubles of a slot; its word's place
  for (int q = 0; q < 2; ++q) *host_word(pin_host + kSlot * q + kWord) = ~0ull;
  long long R = 1, Q = 0, neval = n;
  auto split_size = [&] {
    return std::min<long long>({(long long)sp.nsplit, R, (sp.maxeval - neval) / (2 * n)});
  };
  auto sample = [&](long long nchild) -> int {
    const Pieces p = tile_pieces(n, nchild, fine, ctx->ncu, lds);
    A.tile = p.size;
    A.ntiles = p.count;
    CCUBA_HIP(launch_suave_sample(A, (int)nchild, s));
    CCUBA_HIP(launch_suave_fold(A, (int)nchild, s));
    return CCUBA_OK;
  };
  auto totals = [&](long long t) -> int {
    double *slot = pin_dev + kSlot * (t % 2);
    const SStop stop{sp.epsrel, sp.epsabs, sp.mineval, neval, (unsigned long long)t,
                     (SState *)slot, (unsigned long long *)(slot + kWord),
                     split_size() <= 0 ? 1 : 0, 0};
    CCUBA_HIP(launch_suave_totals(A, (int)R, stop, s));
    return CCUBA_OK;
  };
  // the root region
  CCUBA_HIP(launch_suave_root(A, s));
  if ((rc = sample(1)) || (rc = totals(0))) return rc;
  int fail = 1;
  long long t = 0;
  for (;; ++t) {
    const long long K = split_size();
    if (K > 0) {  // changes no region
      const Pieces p = chunk_pieces(n, K, fine, ctx->ncu);
      A.chunk = p.size;
      A.nchunks = p.count;
      CCUBA_HIP(launch_suave_select(A, (int)R, (int)K, s));
      CCUBA_HIP(launch_suave_fluct(A, (int)K, s));
    }
    const int code = poll_outcome(pin_host + kSlot * (t % 2) + kWord, (unsigned long long)t, s);
    if (code < 0) return code;
    if (code || K <= 0) {
      fail = code == 2 ? -4 : code == 1 ? 0 : 1;
      break;
    }
    CCUBA_HIP(launch_suave_split(A, (int)R, Q, (int)K, s));
    if ((rc = sample(2 * K))) return rc;
    R += K;
    Q += K;
    neval += 2 * K * n;
    if ((rc = totals(t + 1))) return rc;
  }
  CCUBA_HIP(hipStreamSynchronize(s));
  SState st{};
  if (fail != -4) std::memcpy(&st, pin_host + kSlot * (t % 2), sizeof(st));
  res.integral = st.I;
  res.error = std::sqrt(st.var);
  res.prob = st.prob;
  res.chi2 = st.chi2;
  res.dof = st.dof;
  res.fail = fail;
  res.nregions = (int)R;
  res.neval = neval;
  res.nsplits = Q;
  if (tr) {
    const size_t m = (size_t)std::min<long long>(R, tr->max_regions);
    if (m > 0) {
      if (tr->lo) CCUBA_HIP(hipMemcpyAsync(tr->lo, B.lo.p, m * d * 8, hipMemcpyDeviceToHost, s));
      if (tr->hi) CCUBA_HIP(hipMemcpyAsync(tr->hi, B.hi.p, m * d * 8, hipMemcpyDeviceToHost, s));
      if (tr->I) CCUBA_HIP(hipMemcpyAsync(tr->I, B.I.p, m * 8, hipMemcpyDeviceToHost, s));
      if (tr->var) CCUBA_HIP(hipMemcpyAsync(tr->var, B.var.p, m * 8, hipMemcpyDeviceToHost, s));
      if (tr->grid)
        CCUBA_HIP(hipMemcpyAsync(tr->grid, B.grid.p, m * row * 8, hipMemcpyDeviceToHost, s));
    }
    const size_t q = (size_t)std::min<long long>(Q, tr->max_splits);
    if (q > 0 && tr->cut)
      CCUBA_HIP(hipMemcpyAsync(tr->cut, B.cut.p, q * sizeof(int), hipMemcpyDeviceToHost, s));
    CCUBA_HIP(hipStreamSynchronize(s));
  }
  return CCUBA_OK;
}

}  // namespace ccuba
