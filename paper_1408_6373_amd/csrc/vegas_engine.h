// vegas_engine.h -- host driver of the batched Vegas DoSample engine.
//
// One engine holds any number of independent Vegas integrals resident on the
// device (grids, parameters, partial sums, iteration history, state) and
// advances all of them one iteration per launch pair (DoSample + refine).
// A single integral is an engine with one job.
#pragma once
#include <functional>
#include <utility>
#include <vector>

#include "context.h"
#include "vegas.h"

namespace ccuba {

constexpr int kIterCap = 4096;  // iterations kept per integral

// Host description of one Vegas integral.
struct VegasSpec {
  int ndim = 1, nbins = 128, family = 0, prec = FP64, flags = 0;
  unsigned long long seed = 0;
  uint32_t sid = 0;
  long long nstart = 1000, nincrease = 0, mineval = 0, maxeval = 0;
  double epsrel = 0, epsabs = 0;
  double a[kMaxDim] = {0}, u[kMaxDim] = {0};
};

// Validate a spec; CCUBA_OK or CCUBA_EINVAL.
int validate_vegas(const VegasSpec &s);
// Iterations the budget allows and the largest n_t among them.
void vegas_budget(const VegasSpec &s, int *iters, long long *nmax);
// Where a batch splits into two halves of about equal evaluations (the
// budget's iterations): the first `cut' integrals and the rest, each holding
// at least one; specs.size() for fewer than two.
size_t batch_cut(const std::vector<VegasSpec> &specs);
// The per-dimension constants of the device Genz code (see genz.h).
void genz_constants(const VegasSpec &s, double p64[2][kParamRow], float p32[2][kParamRow]);

// A slice of a launch's tile list holding the tiles of every job of one
// (precision, Philox blocks per point) class, with the LDS it needs.
struct TileGroup {
  int prec, nb, pow2, full, first, count;
  size_t grid_bytes, lds;
  int hfx;  // 1: the fixed-point LDS histogram instance
};

// Dynamic LDS of a DoSample instance (the layouts of vegas_sample.h) for an
// integral of dimension d with N bins; *hist_off: where its histogram starts
// when that is not a constant of the instance.
size_t dosample_lds(int prec, bool fixed, int nb, bool pow2, int d, int N, size_t *hist_off);

// Whether the DoSample launch of a class takes the fixed-point LDS histogram:
// unless hist64 asks for the FP64 one, or (FP64 evaluation: 16-byte cells and
// three histogram words per bin) the class's largest d N would not fit the LDS.
bool fixed_hist(int prec, int hist64, long long dN);

// Order the tiles of `jobs' by class, set each job's tile0 to the position of
// its first tile, and describe the classes.  Also returns the refine LDS.
void plan_tile_groups(std::vector<VJob> &jobs, std::vector<int> &tiles,
                      std::vector<TileGroup> &groups, const int hist64[2],
                      size_t *refine_lds);
// One DoSample launch per class; `user' (if given) is the run-time compiled
// kernel of the one class of a caller's device integrand.
int launch_tile_groups(ccuba_ctx *ctx, VegasArgs A, const std::vector<TileGroup> &groups,
                       hipStream_t s, hipFunction_t user = nullptr);
// Inclusive prefixes over jobs of their fold tasks (see FoldArgs).
void fold_tasks(const std::vector<VJob> &jobs, std::vector<long long> &ends, long long *total);
// Blocks of a DoSample instance that a compute unit's LDS holds at once.
int lds_blocks(size_t lds);

// Points of a tile of a single integral (dN = ndim nbins) whose largest iteration
// has n points, a multiple of bs (its block): about one tile per block, of at most
// blocks_per_cu blocks on each of ncu compute units, which hold `resident' at once;
// refined: a refine launch follows.
long long single_tile(long long n, long long bs, int ncu, int blocks_per_cu, int prec,
                      long long dN, int resident, bool refined);

// The same for the integrals of one precision of a batch (of an engine: one or both
// halves), which take total points in their largest iterations, rows the sum of
// their points times d N.
long long batch_tile(long long total, double rows, long long min_tile, long long bs, int ncu,
                     int blocks_per_cu);

// Whether the refine launch can sum every job's tile rows itself (no fold).
bool direct_refine(const std::vector<VJob> &jobs);

class VegasEngine {
 public:
  explicit VegasEngine(ccuba_ctx *ctx) : ctx_(ctx) {}
  // Allocate and upload; `single' plans tiles for one large integral.
  int setup(const std::vector<VegasSpec> &specs, bool single, hipStream_t s);
  // One iteration of every unfinished job (async on s).
  int step(hipStream_t s);
  // Iterate until every job is done; replays a captured graph if enabled.
  // run = launch_run then finish_run.
  int run(hipStream_t s);
  // Capture ahead the graphs that launch_run replays when every job runs
  // its whole budget (nothing to do otherwise), so that launch_run then only
  // queues them.
  int prepare_run(hipStream_t s);
  // Launch the iterations: all without waiting when every job runs its
  // whole budget (fixed()); else in chunks with host checks of the states, or
  // (one integral, set_alone) one at a time, one ahead of the last whose
  // outcome the host has polled.
  int launch_run(hipStream_t s);
  // Wait for everything queued on the engine's stream.
  int drain(hipStream_t s);
  // Wait for what launch_run queued; the profile-mode timings.
  int finish_run(hipStream_t s);
  // No job can stop before its budget (no epsrel or epsabs).
  bool fixed() const;
  // The same one iteration at a time, calling after(state of job 0) once each
  // iteration is done (a checkpoint); a nonzero return from it stops the run
  // with that status.
  int run_each(hipStream_t s, const std::function<int(const VState &)> &after);
  // Job 0 continues from a saved state, grid and history (T = st.T
  // iterations done); call after setup.
  int load_checkpoint(const VState &st, const double *grid, const double *I, const double *var,
                      hipStream_t s);
  // Job 0's history capacity (iterations the budget allows).
  int hist_cap() const { return hjobs_.empty() ? 0 : hjobs_[0].hist_cap; }
  // Job 0's state, its history (the first max_iter iterations at most) and its
  // grid, where given, once the stream has drained (through the context's
  // pinned block).
  int read_results(VState &st, double *I, double *var, int max_iter, double *grid,
                   hipStream_t s);
  int read_states(std::vector<VState> &out, hipStream_t s);
  int read_grid(int job, double *grid, hipStream_t s);
  // The grid and iteration t's estimate and variance of one job, read with
  // one synchronisation (what a checkpoint needs after each iteration).
  int read_step(int job, int t, double *grid, double *I, double *var, hipStream_t s);
  // Raw pieces: set iteration index of job 0, run DoSample only.
  int set_iteration(int job, int t, hipStream_t s);
  int load_grid(int job, const double *src, hipMemcpyKind kind, hipStream_t s);
  // the sampling kernels, then the fold (both levels, into the one job's sums
  // and hist where they are given; else only where the refine launch needs
  // it); records `between` (if given) after the sampling kernels
  int dosample_only(hipStream_t s, hipEvent_t between = nullptr, double *sums = nullptr,
                    double *hist = nullptr);
  // One refinement of job 0 from a given histogram and grid.
  int refine_only(const double *hist, const double *grid_in, double *grid_out, hipStream_t s);

  // The caller runs this engine alone on the context, so that its run may use
  // the context's pinned block (launch_polled).
  void set_alone() { alone_ = true; }
  // The engine runs once and is not kept: its launches are queued one by one, as
  // capturing and instantiating a graph of them costs more than it saves.  10
  // iterations of 10^5 points at d = 8: 212 us; 271 with a graph, and 406 in half
  // of the processes.
  void set_once() { once_ = true; }
  // The engine makes sampling passes only (dosample_only with sums); before setup.
  void set_raw() { raw_ = true; }
  // A caller's device integrand (family USER): its compiled DoSample kernel,
  // set before setup.
  void set_user_kernel(hipFunction_t f) { user_fn_ = f; }

  // Profile mode with a reference event recorded before this engine's work
  // (on its stream or one it waits on): each iteration's sampling interval,
  // in ms after the reference, goes to dosample_intervals() instead of the
  // context's busy time, so that a caller running engines side by side can
  // take the union.
  void set_time_reference(hipEvent_t ref) { ref_ = ref; }
  const std::vector<std::pair<double, double>> &dosample_intervals() const { return ds_iv_; }

  int njobs() const { return (int)specs_.size(); }
  int max_iters() const { return max_iters_; }
  long long evals_per_iteration() const { return evals_iter_; }
  const std::vector<VegasSpec> &specs() const { return specs_; }
  // launch geometry actually used
  int grid_blocks(int prec) const { return nblocks_[prec]; }
  int block() const { return block_[1]; }

 private:
  int launch_iteration(hipStream_t s);
  int launch_polled(hipStream_t s);
  int flush_timing();
  struct Timed {
    hipEvent_t e0, e1, e2, e3;
    int iter;
  };
  std::vector<Timed> pending_;
  hipEvent_t ref_ = nullptr;
  std::vector<std::pair<double, double>> ds_iv_;
  bool capturing_ = false, alone_ = false, once_ = false, raw_ = false;
  hipStream_t busy_ = nullptr;  // the stream that may still hold the engine's work
  int iter_launched_ = 0;
  ccuba_ctx *ctx_;
  std::vector<VegasSpec> specs_;
  std::vector<VJob> hjobs_;
  DevBuf<VJob> jobs_;
  DevBuf<VState> state_;
  DevBuf<int> tile_job_;
  DevBuf<double> grids_, p64_, tile_sums_, tile_hist_, group_sums_, group_hist_, iter_I_,
      iter_var_;
  DevBuf<float> p32_;
  DevBuf<long long> fold_end_;
  long long fold_total_ = 0;
  VegasArgs args_{};
  bool direct_ = false;  // the refine launch sums the tile rows (direct_refine)
  int ntiles_ = 0, ngroups_ = 0;
  std::vector<TileGroup> tgroups_;
  int has_prec_[2] = {0, 0};
  int nblocks_[2] = {0, 0}, block_[2] = {256, 256};
  size_t lds_refine_ = 0;
  int hist64_[2] = {0, 0};  // per precision: the FP64 LDS histogram asked for
  hipFunction_t user_fn_ = nullptr;
  int max_iters_ = 0;
  int dmax_ = 1;  // the largest dimension among the jobs (refine launch)
  long long evals_iter_ = 0;
  // instantiated graphs of k consecutive iterations
  struct ChunkGraph {
    int k;
    hipGraphExec_t exec;
  };
  std::vector<ChunkGraph> graphs_;
  std::vector<long long> graph_sig_;  // the launch arguments the graphs hold
  static constexpr int kMaxGraphIters = 32;
  int graph_for(int k, hipStream_t s, hipGraphExec_t *out);

 public:
  ~VegasEngine();
};

}  // namespace ccuba
