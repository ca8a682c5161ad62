// divonne.hip -- Divonne's partitioning phase on gfx950 (Sect. 2.2).
//
// Spread(r) = 1/2 Vol(r) (sup_r f - inf_r f).  One step:
//   topk    the K regions of largest spread (the Suave selection kernel)
//   split   per selected region, one wavefront: d probes f(xmax with
//           x_j := xmin_j); the cut goes through the midpoint of the
//           dimension of largest loss fmax - f_j; the two children
//   search  per child: two wavefronts evaluate its nsearch Philox points and
//           reduce to the largest and smallest value (ties to the lower
//           index); then one group of lanes climbs to the maximum and one
//           descends to the minimum by compass search, lane c < 2d of a group
//           evaluating candidate c (x +- h_j e_j, clipped) each iteration; a
//           move is taken when the best candidate (ties to the lower c) beats
//           the current value, else every step halves
//   totals  the largest and the total spread over all regions (fixed order)
// The selection changes no region, so the host learns a step's outcome while
// the next one's runs.
#include "divonne.h"
#include "genz.h"
#include "philox.h"

namespace ccuba {

namespace {

template <int FAM>
__device__ __forceinline__ double eval_at(const double *x, int d, const double *p0,
                                          const double *p1) {
  double acc = Genz<double, FAM>::init(p1[0]);
  for (int j = 0; j < d; ++j) acc = Genz<double, FAM>::step(acc, x[j], p0[j], p1[j]);
  return Genz<double, FAM>::finish(acc, d);
}

// one DPP step of the reduction below: each lane compares itself with the
// lane the control selects (lanes without a source compare with themselves)
template <int CTRL, int ROWS, int BANKS>
__device__ __forceinline__ void best_step(double &v, int &idx, double sign) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp((int)b, (int)b, CTRL, ROWS, BANKS, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), CTRL, ROWS, BANKS,
                                             false);
  const int oi = __builtin_amdgcn_update_dpp(idx, idx, CTRL, ROWS, BANKS, false);
  const double ov = __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
  if (sign * ov > sign * v || (ov == v && oi < idx)) {
    v = ov;
    idx = oi;
  }
}

// (value, index) reduction over a wavefront: the larger sign*value, ties to
// the lower index; every lane gets the winner.  "Best of" is idempotent, so
// the DPP pattern may count a lane twice: row shifts by 1, 2, 4 and 8 leave
// each row's best in its lane 15, the row broadcasts carry it to lane 63,
// whose result readlane hands to every lane.
__device__ __forceinline__ void wave_best(double &v, int &idx, double sign) {
  best_step<0x111, 0xf, 0xf>(v, idx, sign);  // row_shr:1
  best_step<0x112, 0xf, 0xf>(v, idx, sign);  // row_shr:2
  best_step<0x114, 0xf, 0xf>(v, idx, sign);  // row_shr:4
  best_step<0x118, 0xf, 0xf>(v, idx, sign);  // row_shr:8
  best_step<0x142, 0xa, 0xf>(v, idx, sign);  // row_bcast:15 into rows 1 and 3
  best_step<0x143, 0xc, 0xf>(v, idx, sign);  // row_bcast:31 into rows 2 and 3
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, 63);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
  v = __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
  idx = __builtin_amdgcn_readlane(idx, 63);
}

}  // namespace

__global__ void __launch_bounds__(64) div_root_kernel(DivArgs A) {
  if (threadIdx.x < A.d) {
    A.R.lo[threadIdx.x] = 0.0;
    A.R.hi[threadIdx.x] = 1.0;
  }
  if (threadIdx.x == 0) {
    A.chpos[0] = 0;
    A.chser[0] = 0;
  }
}

namespace {

// the lane values a row rotation by CTRL - 0x120 lanes brings (rows of 16)
template <int CTRL>
__device__ __forceinline__ double row_ror(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// the largest value of each group of GL = 16 or 32 lanes, in all its lanes
// (NaNs lose)
template <int GL>
__device__ __forceinline__ double group_max(double v) {
  v = fmax(v, row_ror<0x128>(v));
  v = fmax(v, row_ror<0x124>(v));
  v = fmax(v, row_ror<0x122>(v));
  v = fmax(v, row_ror<0x121>(v));
  if constexpr (GL == 32) v = fmax(v, __shfl_xor(v, 16, 64));
  return v;
}

}  // namespace

// A search has 2d candidates an iteration, so it takes a group of 16 lanes
// (d <= 8) or 32, and one wavefront climbs for two regions' maxima and minima
// at once, or one's: a wavefront per search leaves 3/4 of its lanes idle at
// d = 8.  The search sample has a block's two wavefronts per region.
template <int NB>
struct DivShape {
  static constexpr int kGroup = NB <= 2 ? 16 : 32;       // lanes of one search
  static constexpr int kRegions = 64 / (2 * kGroup);     // regions of a block
  static constexpr int kThreads = kDivBlock * kRegions;  // two wavefronts a region
};

// What bounds it: the chain of niter dependent iterations of a region (small
// launches), instruction issue with about one wavefront per SIMD (large
// ones).  D = 4 NB coordinates in registers (d <= D): the point lives in every
// lane of a group; a lane's own coordinate, its step and its bounds are held
// apart, so that an iteration selects nothing by a lane-varying index.  The
// best candidate is a row-rotation maximum and a ballot; ties go to the lower
// candidate.  Gaussian d = 8, 1024 search points and 64 iterations, launches of
// 1 to 2048 regions on the way to 8192: 42.2 us a launch on average, 90.9 with a
// wavefront per search, lane-varying selects and a six-step (value, index)
// reduction.
template <int FAM, int NB>
__global__ void __launch_bounds__(DivShape<NB>::kThreads) div_search_kernel(DivArgs A,
                                                                            int nchild) {
  constexpr int D = 4 * NB, GL = DivShape<NB>::kGroup, RB = DivShape<NB>::kRegions;
  __shared__ double sLo[RB][kMaxDim], sW[RB][kMaxDim];
  __shared__ double sv[2 * RB][2];
  __shared__ int si[2 * RB][2];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, d = A.d;
  const int first = blockIdx.x * RB;
  // (an odd launch's last block searches its one region twice and writes once)
  if (tid < RB * kMaxDim && tid % kMaxDim < d) {
    const int r = tid / kMaxDim, j = tid % kMaxDim;
    const int pos = A.chpos[min(first + r, nchild - 1)];
    const double lo = A.R.lo[(size_t)pos * d + j];
    sLo[r][j] = lo;
    sW[r][j] = A.R.hi[(size_t)pos * d + j] - lo;
  }
  __syncthreads();
  // Coordinates from d to D are 0 with constants that leave every family's
  // running value as it is (a factor 0 of a sum's term, a factor 1 of the
  // product peak), so that no step tests j < d.
  double p0[D], p1[D];  // (the rows are zero-padded)
#pragma unroll
  for (int j = 0; j < D; ++j) {
    p0[j] = FAM == PRODUCT_PEAK && j >= d ? 1.0 : A.p64[j];
    p1[j] = A.p64[kParamRow + j];
  }
  // the point of search-sample index i of the region with search serial q
  auto point = [&](int i, int q, const double *lo, const double *wd, double (&x)[D]) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const U4 W = philox4x32_10(U4{(uint32_t)i, ((uint32_t)q << 8) | (uint32_t)b, A.sid, 0u},
                                 A.key0, A.key1);
      const uint32_t r[4] = {W.x, W.y, W.z, W.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int j = 4 * b + k;
        x[j] = j < d ? fma((double)r[k] * 0x1p-32 + 0x1p-33, wd[j], lo[j]) : 0.0;
      }
    }
  };
  // the search sample: wavefronts 2r and 2r + 1 take region r's points
  {
    const int r = w >> 1, t = tid & (kDivBlock - 1);
    const int q = A.chser[min(first + r, nchild - 1)];
    double lo[D], wd[D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
      lo[j] = j < d ? sLo[r][j] : 0.0;
      wd[j] = j < d ? sW[r][j] : 0.0;
    }
    double bmax = -INFINITY, bmin = INFINITY;
    int imax = 0x7fffffff, imin = 0x7fffffff;
    for (int i = t; i < A.nsearch; i += kDivBlock) {
      double x[D];
      point(i, q, lo, wd, x);
      double acc = Genz<double, FAM>::init(p1[0]);
#pragma unroll
      for (int j = 0; j < D; ++j) acc = Genz<double, FAM>::step(acc, x[j], p0[j], p1[j]);
      const double f = Genz<double, FAM>::finish(acc, d);
      if (f > bmax) {  // i grows, so a tie keeps the lower index
        bmax = f;
        imax = i;
      }
      if (f < bmin) {
        bmin = f;
        imin = i;
      }
    }
    wave_best(bmax, imax, 1.0);
    wave_best(bmin, imin, -1.0);
    if (lane == 0) {
      sv[w][0] = bmax;
      si[w][0] = imax;
      sv[w][1] = bmin;
      si[w][1] = imin;
    }
  }
  __syncthreads();
  if (w != 0) return;
  // one wavefront from here: group g searches region g / 2's maximum (even g)
  // or minimum (odd g), from the sample's best
  const int g = lane / GL, c = lane & (GL - 1), base = lane & ~(GL - 1);
  const int r = g >> 1, k = g & 1;
  const bool write = first + r < nchild;
  const int child = min(first + r, nchild - 1);
  const int pos = A.chpos[child];
  const double sign = k == 0 ? 1.0 : -1.0;
  double sfx;  // sign * (the value held)
  int i0;
  {
    const double v0 = sign * sv[2 * r][k], v1 = sign * sv[2 * r + 1][k];
    const int j0 = si[2 * r][k], j1 = si[2 * r + 1][k];
    const bool second = v1 > v0 || (v1 == v0 && j1 < j0);
    sfx = second ? v1 : v0;
    i0 = second ? j1 : j0;
  }
  double x[D];
  point(i0, A.chser[child], sLo[r], sW[r], x);
  // lane c < 2d owns candidate c: coordinate jc = c/2, + for even c
  const int jc = c >> 1;
  const bool plus = (c & 1) == 0, live = c < 2 * d;
  const double loj = live ? sLo[r][jc] : 0.0, wj = live ? sW[r][jc] : 0.0;
  const double hij = loj + wj;
  double hj = wj / 4.0, xj = 0.0;
#pragma unroll
  for (int j = 0; j < D; ++j)
    if (j == jc) xj = x[j];
  for (int t = 0; t < A.niter; ++t) {
    const double zc = fmin(fmax(plus ? xj + hj : xj - hj, loj), hij);
    double acc = Genz<double, FAM>::init(p1[0]);
#pragma unroll
    for (int j = 0; j < D; ++j)
      acc = Genz<double, FAM>::step(acc, j == jc ? zc : x[j], p0[j], p1[j]);
    const double sf = live ? sign * Genz<double, FAM>::finish(acc, d) : -INFINITY;
    const double best = group_max<GL>(sf);
    const uint32_t eq = (uint32_t)(__ballot(live && sf == best) >> base) &
                        (uint32_t)((1ull << GL) - 1ull);
    const int win = __ffs((int)eq) - 1;  // (-1 when every candidate is NaN: no move then)
    const double znew = __shfl(zc, base + max(win, 0), 64);
    const bool move = best > sfx;
    const int jw = move ? win >> 1 : -1;
    sfx = move ? best : sfx;
    xj = jc == jw ? znew : xj;
    hj = move ? hj : hj * 0.5;
#pragma unroll
    for (int j = 0; j < D; ++j) x[j] = j == jw ? znew : x[j];
  }
  const double fx = sign * sfx, other = __shfl_xor(fx, GL, 64);
  if (!write) return;
  if (live && plus) (k == 0 ? A.R.xmax : A.R.xmin)[(size_t)pos * d + jc] = xj;
  if (c == 0) {
    (k == 0 ? A.R.fmax : A.R.fmin)[pos] = fx;
    if (k == 0) {
      double V = 1.0;
      for (int j = 0; j < d; ++j) V *= sW[r][j];
      A.R.spread[pos] = 0.5 * V * (fx - other);
    }
  }
}

// Per selected region (one wavefront): the cut and the two children.
template <int FAM>
__global__ void __launch_bounds__(64) div_split_kernel(DivArgs A, int R, long long Q) {
  __shared__ double sXmax[kMaxDim], sXmin[kMaxDim], sP0[kMaxDim], sP1[kMaxDim];
  const int s = blockIdx.x, lane = threadIdx.x, d = A.d;
  const int pos = A.sel[s], up = R + s;
  if (lane < d) {
    sXmax[lane] = A.R.xmax[(size_t)pos * d + lane];
    sXmin[lane] = A.R.xmin[(size_t)pos * d + lane];
    sP0[lane] = A.p64[lane];
    sP1[lane] = A.p64[kParamRow + lane];
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const double fmax = A.R.fmax[pos];
  double loss = -INFINITY;
  int idx = 0x7fffffff;
  if (lane < d) {
    double acc = Genz<double, FAM>::init(sP1[0]);
    for (int j = 0; j < d; ++j)
      acc = Genz<double, FAM>::step(acc, j == lane ? sXmin[j] : sXmax[j], sP0[j], sP1[j]);
    loss = fmax - Genz<double, FAM>::finish(acc, d);
    idx = lane;
  }
  wave_best(loss, idx, 1.0);
  const int c = idx;
  if (lane < d) {
    const double lo = A.R.lo[(size_t)pos * d + lane], hi = A.R.hi[(size_t)pos * d + lane];
    const double mid = 0.5 * (lo + hi);
    A.R.lo[(size_t)up * d + lane] = lane == c ? mid : lo;
    A.R.hi[(size_t)up * d + lane] = hi;
    if (lane == c) A.R.hi[(size_t)pos * d + lane] = mid;
  }
  if (lane == 0) {
    A.cut[Q + s] = c;
    A.chpos[2 * s] = pos;
    A.chpos[2 * s + 1] = up;
    A.chser[2 * s] = (int)(2 * (Q + s) + 1);
    A.chser[2 * s + 1] = (int)(2 * (Q + s) + 2);
  }
}

// The largest and the total spread over the R regions (fixed order), and the
// stop rule's outcome as one word, seq << 8 | code, that the host polls (code
// 0: go on, 1: every spread within spread_tol, 2: not finite).
__global__ void __launch_bounds__(1024) div_totals_kernel(DivArgs A, int R, DStop stop) {
  __shared__ double rs[16], rm[16];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int chunk = (R + 1023) / 1024;
  const int b0 = min(tid * chunk, R), b1 = min(b0 + chunk, R);
  double sum = 0.0, mx = 0.0;
  for (int i = b0; i < b1; ++i) {
    const double v = A.R.spread[i];
    sum += v;
    mx = fmax(mx, v);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    sum += __shfl_xor(sum, o, 64);
    mx = fmax(mx, __shfl_xor(mx, o, 64));
  }
  if (lane == 0) {
    rs[w] = sum;
    rm[w] = mx;
  }
  __syncthreads();
  if (tid == 0) {
    double S = 0.0, M = 0.0;
    for (int q = 0; q < 16; ++q) {
      S += rs[q];
      M = fmax(M, rm[q]);
    }
    stop.state->max_spread = M;
    stop.state->total_spread = S;
    const unsigned long long code = !isfinite(S) ? 2u : M <= stop.spread_tol ? 1u : 0u;
    __hip_atomic_store(stop.word, (stop.seq << 8) | code, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// ---- launchers ---------------------------------------------------------------

hipError_t launch_div_root(const DivArgs &A, hipStream_t s) {
  hipLaunchKernelGGL(div_root_kernel, dim3(1), dim3(64), 0, s, A);
  return hipGetLastError();
}

#define CCUBA_DIV_FAMILY_SWITCH(KERNEL, GRID, BLOCK, ...)                               \
  switch (A.family) {                                                                   \
    case GAUSSIAN:                                                                      \
      hipLaunchKernelGGL(KERNEL<GAUSSIAN>, GRID, BLOCK, 0, s, __VA_ARGS__);             \
      break;                                                                            \
    case OSCILLATORY:                                                                   \
      hipLaunchKernelGGL(KERNEL<OSCILLATORY>, GRID, BLOCK, 0, s, __VA_ARGS__);          \
      break;                                                                            \
    case PRODUCT_PEAK:                                                                  \
      hipLaunchKernelGGL(KERNEL<PRODUCT_PEAK>, GRID, BLOCK, 0, s, __VA_ARGS__);         \
      break;                                                                            \
    case CORNER_PEAK:                                                                   \
      hipLaunchKernelGGL(KERNEL<CORNER_PEAK>, GRID, BLOCK, 0, s, __VA_ARGS__);          \
      break;                                                                            \
    default:                                                                            \
      hipLaunchKernelGGL(KERNEL<C0>, GRID, BLOCK, 0, s, __VA_ARGS__);                   \
      break;                                                                            \
  }

template <int NB>
static void launch_search_nb(const DivArgs &A, int nchild, hipStream_t s) {
  constexpr int RB = DivShape<NB>::kRegions;
  const dim3 grid((nchild + RB - 1) / RB), block(DivShape<NB>::kThreads);
  switch (A.family) {
    case GAUSSIAN:
      hipLaunchKernelGGL((div_search_kernel<GAUSSIAN, NB>), grid, block, 0, s, A, nchild);
      break;
    case OSCILLATORY:
      hipLaunchKernelGGL((div_search_kernel<OSCILLATORY, NB>), grid, block, 0, s, A, nchild);
      break;
    case PRODUCT_PEAK:
      hipLaunchKernelGGL((div_search_kernel<PRODUCT_PEAK, NB>), grid, block, 0, s, A, nchild);
      break;
    case CORNER_PEAK:
      hipLaunchKernelGGL((div_search_kernel<CORNER_PEAK, NB>), grid, block, 0, s, A, nchild);
      break;
    default:
      hipLaunchKernelGGL((div_search_kernel<C0, NB>), grid, block, 0, s, A, nchild);
      break;
  }
}

hipError_t launch_div_search(const DivArgs &A, int nchild, hipStream_t s) {
  switch ((A.d + 3) / 4) {
    case 1:
      launch_search_nb<1>(A, nchild, s);
      break;
    case 2:
      launch_search_nb<2>(A, nchild, s);
      break;
    case 3:
      launch_search_nb<3>(A, nchild, s);
      break;
    default:
      launch_search_nb<4>(A, nchild, s);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_div_split(const DivArgs &A, int R, long long Q, int K, hipStream_t s) {
  CCUBA_DIV_FAMILY_SWITCH(div_split_kernel, dim3(K), dim3(64), A, R, Q)
  return hipGetLastError();
}

#undef CCUBA_DIV_FAMILY_SWITCH

hipError_t launch_div_totals(const DivArgs &A, int R, const DStop &stop, hipStream_t s) {
  hipLaunchKernelGGL(div_totals_kernel, dim3(1), dim3(1024), 0, s, A, R, stop);
  return hipGetLastError();
}

}  // namespace ccuba
