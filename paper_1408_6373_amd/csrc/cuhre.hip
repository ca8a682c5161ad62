// cuhre.hip -- Cuhre on gfx950: the degree-7 Genz-Malik rule over batches of
// subregions, top-K selection, bisection and compaction of the region heap.
//
// a8 (the DoSample of Cuhre): one wavefront per region (one workgroup in
//    small launches, one lane at small d in large ones).  The lanes walk the
//    2^d + 2d^2 + 2d + 1 rule points (Genz & Malik 1980) of their region,
//    decoding each point index to its generator class and axes, evaluate the
//    Genz integrand in FP64, and keep five class sums; the class-2 and
//    class-3 values and the centre go to LDS for the fourth differences.
//    Wave shuffles reduce the class sums; lane 0 forms
//      I7 = prod(h) sum_k w7_k S_k,  I5 = prod(h) sum_k w5_k S_k,
//      err = |I7 - I5|,
//    and the lanes j < d form the fourth difference
//      D_j = |f(c+l2 h_j e_j) + f(c-l2 h_j e_j) - 2 f(c)
//             - (l2^2/l3^2)(f(c+l3 h_j e_j) + f(c-l3 h_j e_j) - 2 f(c))|,
//    whose arg-max (lowest j on ties) is the split axis.  A launch takes a
//    list of segments, so regions of several integrals share one launch.
// a9 (region step): the store of regions only grows (a region's position is
//    its id) and a split region is retired in place.  Selection of the K
//    largest errors by a 16-bit digit histogram and an exact rank within the
//    boundary digit (ties go to the lower position, i.e. the lower region
//    id); a counting pass and a scan give each selected region its rank j,
//    and the rule launch forms the two halves of the j-th at the end of the
//    store before it evaluates them; a fixed-order reduction gives the
//    totals.  Where a step needs the whole grid's results (a scan of block
//    counts, a reduction of block sums, a pick from the histogram), a
//    one-workgroup kernel follows: no block ever waits for another, and no
//    block fences for another (a device-scope release writes back the L2
//    of its XCD, ~0.7 us each, serialised per XCD, which costs more per
//    block than a kernel boundary costs once).
#include <algorithm>

#include "cuhre.h"
#include "genz.h"
#include "vegas_sample.h"  // uniform
#include "wave.h"

namespace ccuba {

namespace {

// The rule's weights per dimension (rows 0..16): degree 7 and degree 5.
struct GMWeights {
  double w7[17 * 5], w5[17 * 5];
};
constexpr GMWeights gm_weights() {
  GMWeights t{};
  for (int d = 0; d <= 16; ++d) {
    const double p2 = (double)(1 << d), dd = d;
    double *w7 = t.w7 + 5 * d, *w5 = t.w5 + 5 * d;
    w7[0] = p2 * (12824.0 - 9120.0 * dd + 400.0 * dd * dd) / 19683.0;
    w7[1] = p2 * 980.0 / 6561.0;
    w7[2] = p2 * (1820.0 - 400.0 * dd) / 19683.0;
    w7[3] = p2 * 200.0 / 19683.0;
    w7[4] = 6859.0 / 19683.0;
    w5[0] = p2 * (729.0 - 950.0 * dd + 50.0 * dd * dd) / 729.0;
    w5[1] = p2 * 245.0 / 486.0;
    w5[2] = p2 * (265.0 - 100.0 * dd) / 1458.0;
    w5[3] = p2 * 25.0 / 729.0;
    w5[4] = 0.0;
  }
  return t;
}
__constant__ GMWeights kWeights = gm_weights();

constexpr int kLaneRuleMaxDim = 8;          // lane-per-region rule up to this d
constexpr long long kLaneRuleMinRegions = 512;  // and from this many regions on
constexpr long long kOneLaneRuleMinRegions = 49152;  // one lane per region from here
// Whether it may: a lane holds the unrolled pairs and the corners' tree, and around
// a cosine, whose own registers come on top, they spill from d = 4 on (a lane of
// four wavefronts holds a quarter of them).  4 x 10^5 regions, oscillatory, us:
//   d       4    5    6    7     8
//   one   112  213  475  755  1039
//   four   95  156  235  411   613
constexpr bool one_lane_rule(int family, int d) { return family != OSCILLATORY || d < 4; }
constexpr long long kWaveRuleBlocks = 2048;       // most blocks of a wave-per-region launch
// Up to this many regions a launch over several integrals or above 8
// dimensions gives each a whole workgroup (its four wavefronts share the rule
// points): about what the device holds at once, so that the launch takes as
// long as one region does.
constexpr long long kBlockRuleRegions = 1024;
constexpr int kScanItems = 4;
constexpr int kScanBlock = 256;
constexpr int kScanTile = kScanItems * kScanBlock;  // elements per scan block

__device__ __forceinline__ double wsum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Selection key of a region: the IEEE bit pattern of its error plus one,
// which orders the non-negative doubles; 0 for a retired region (negative
// error), below every live one.
__device__ __forceinline__ unsigned long long key_of(double e) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(e);
  return (b >> 63) ? 0ull : b + 1ull;
}

__device__ __forceinline__ bool retired(double e) { return signbit(e); }

// The selection's digits are the keys' top 16 bits (sign, exponent and 4
// mantissa bits) in a window of kTopBins values that ends just above the
// digit of the errors' sum E, which no error can exceed: all errors down to
// 2^-255 of the sum have a digit of their own, and smaller ones share digit 0.
__host__ __device__ inline int key_window(double E) {
  unsigned long long b;
  __builtin_memcpy(&b, &E, sizeof(b));
  const long long top = (long long)((b + 1ull) >> 48) + 2;
  return (int)(top > kTopBins ? top - kTopBins : 0);
}
__device__ __forceinline__ int window_digit(unsigned long long key, int base) {
  const int d = (int)(key >> 48) - base;
  return d < 0 ? 0 : d < kTopBins ? d : kTopBins - 1;
}

// The geometry of region r of a segment: loaded, or formed from its parent
// (children mode) and stored.  Lane `j' (< d) handles coordinate j.
__device__ __forceinline__ void child_coord(const CSeg &S, long long r, int j, double *cj,
                                            double *hj) {
  const long long cap = S.regs.cap;
  if (!S.children) {
    *cj = S.regs.c[j * cap + r];
    *hj = S.regs.h[j * cap + r];
    return;
  }
  const long long k = r - S.first;
  const long long p = S.parent ? S.parent[k >> 1] : S.pbase + (k >> 1);
  double c = S.regs.c[j * cap + p], h = S.regs.h[j * cap + p];
  if (j == S.regs.axis[p]) {
    h = h / 2.0;
    c = (k & 1) ? c + h : c - h;
  }
  S.regs.c[j * cap + r] = c;
  S.regs.h[j * cap + r] = h;
  if (S.retire && j == 0 && !(k & 1)) S.regs.err[p] = -1.0;
  *cj = c;
  *hj = h;
}

// Evaluate the Genz family FAM at the rule point described by (cls, i, jj,
// sgn): class 0 centre; 1 and 2: axis i with sign bit 0; 3: axes i < jj with
// sign bits 0 (i) and 1 (jj); 4: every axis, sign bit j for axis j.
template <int FAM>
__device__ __forceinline__ double rule_point_f(int d, const double *c, const double *h,
                                               const double *p0, const double *p1, int cls,
                                               int i, int jj, unsigned sgn, double lam,
                                               double phase0) {
  double acc = Genz<double, FAM>::init(phase0);
  for (int j = 0; j < d; ++j) {
    double x = c[j];
    bool on;
    bool neg;
    if (cls == 4) {
      on = true;
      neg = (sgn >> j) & 1u;
    } else if (cls == 3) {
      on = (j == i) || (j == jj);
      neg = (j == i) ? (sgn & 1u) : ((sgn >> 1) & 1u);
    } else {
      on = (cls != 0) && (j == i);
      neg = sgn & 1u;
    }
    if (on) {
      const double t = lam * h[j];
      x = neg ? x - t : x + t;
    }
    acc = Genz<double, FAM>::step(acc, x, p0[j], p1[j]);
  }
  return Genz<double, FAM>::finish(acc, d);
}

// Order the LDS traffic of the W wavefronts that share a region.
template <int W>
__device__ __forceinline__ void sync_region() {
  if constexpr (W == 1) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// LDS of one region.
struct RuleLds {
  double c[kMaxDim], h[kMaxDim];
  double f[4 * kMaxDim + 1];  // class 1 values, class 2 values, the centre
  double x[2 * kMaxDim];      // c + l5 h and c - l5 h per axis
};

// The class sums over the rule points that thread tid of NT = 2^LB takes, into
// Sk; the class-1 and class-2 values and the centre's to L.f.  p0 and p1 are
// the integrand's constants.
//
// Corners (class 4, all of the work at large d): a thread's low bits fix the
// signs of the first axes, whose part of the integrand's running value is
// formed once; the corners over the remaining axes are the leaves of a tree
// whose last three levels are unrolled, so that a corner costs two to three
// steps and not d (with every step in axis order, as rule_point_f takes them).
// Requests of the serving loop up to d = 16: 15 us a launch, 107 with d steps a
// corner and a wavefront per region.
template <int FAM>
__device__ __forceinline__ void rule_points(const RuleLambdas &A, int d, int tid, int NT, int LB,
                                            RuleLds &L, const double *p0, const double *p1,
                                            double (&Sk)[5]) {
  const double *c = L.c, *h = L.h;
  const double phase0 = p1[0];
  const int n2 = 2 * d, n4 = 2 * d * (d - 1);
  const int b2 = 1, b3 = 1 + n2, b4 = 1 + 2 * n2, b5 = 1 + 2 * n2 + n4;
  // classes 0-3 (a few hundred points at most)
  for (int p = tid; p < b5; p += NT) {
    int cls, i = 0, jj = 0;
    unsigned sgn = 0;
    double lam = 0.0;
    if (p == 0) {
      cls = 0;
    } else if (p < b3) {
      cls = 1;
      i = (p - b2) >> 1;
      sgn = (unsigned)((p - b2) & 1);
      lam = A.l2;
    } else if (p < b4) {
      cls = 2;
      i = (p - b3) >> 1;
      sgn = (unsigned)((p - b3) & 1);
      lam = A.l3;
    } else {
      cls = 3;
      int q = (p - b4) >> 2;
      sgn = (unsigned)((p - b4) & 3);
      i = 0;
      int row = d - 1;
      while (q >= row) {
        q -= row;
        ++i;
        --row;
      }
      jj = i + 1 + q;
      lam = A.l4;
    }
    const double f = rule_point_f<FAM>(d, c, h, p0, p1, cls, i, jj, sgn, lam, phase0);
#pragma unroll
    for (int k = 0; k < 4; ++k) Sk[k] += k == cls ? f : 0.0;
    if (cls == 0) L.f[4 * kMaxDim] = f;
    if (cls == 1) L.f[p - b2] = f;                // [2i + sign]
    if (cls == 2) L.f[2 * kMaxDim + p - b3] = f;  // [2d.. + 2i + sign]
  }
  const int pre = min(LB, d), rest = d - pre;
  if (tid < (1 << pre)) {
    double acc0 = Genz<double, FAM>::init(phase0);
    for (int j = 0; j < pre; ++j)
      acc0 = Genz<double, FAM>::step(acc0, L.x[2 * j + ((tid >> j) & 1)], p0[j], p1[j]);
    // corners over the axes [pre, d), the low bits of m first
    const int mid = rest >= 3 ? rest - 3 : rest;
    double x3[6], q0[3], q1[3];
    if (rest >= 3) {
#pragma unroll
      for (int q = 0; q < 6; ++q) x3[q] = L.x[2 * (d - 3) + q];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        q0[q] = p0[d - 3 + q];
        q1[q] = p1[d - 3 + q];
      }
    }
    for (unsigned m = 0; m < (1u << mid); ++m) {
      double a = acc0;
      for (int q = 0; q < mid; ++q)
        a = Genz<double, FAM>::step(a, L.x[2 * (pre + q) + ((m >> q) & 1u)], p0[pre + q],
                                    p1[pre + q]);
      if (rest < 3) {
        Sk[4] += Genz<double, FAM>::finish(a, d);
        continue;
      }
#pragma unroll 1  // (four corners in flight: eight cost 60 registers more)
      for (int e0 = 0; e0 < 2; ++e0) {
        const double a0 = Genz<double, FAM>::step(a, e0 ? x3[1] : x3[0], q0[0], q1[0]);
#pragma unroll
        for (int e1 = 0; e1 < 2; ++e1) {
          const double a1 = Genz<double, FAM>::step(a0, x3[2 + e1], q0[1], q1[1]);
#pragma unroll
          for (int e2 = 0; e2 < 2; ++e2)
            Sk[4] += Genz<double, FAM>::finish(
                Genz<double, FAM>::step(a1, x3[4 + e2], q0[2], q1[2]), d);
        }
      }
    }
  }
}

// The split axis of the region whose point values are in f: the arg-max of
// the fourth differences, the lowest axis on ties (every lane below 16).
__device__ __forceinline__ int rule_axis(const RuleLambdas &A, int d, int lane, const double *f) {
  double D = -1.0;
  if (lane < d) {
    const double f0 = f[4 * kMaxDim];
    const double a2 = f[2 * lane] + f[2 * lane + 1] - 2.0 * f0;
    const double a3 = f[2 * kMaxDim + 2 * lane] + f[2 * kMaxDim + 2 * lane + 1] - 2.0 * f0;
    const double ratio = (A.l2 * A.l2) / (A.l3 * A.l3);
    D = fabs(a2 - ratio * a3);
  }
  int best = lane;
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {  // (lanes below 16 hold every axis)
    const double oD = __shfl_xor(D, o, 64);
    const int ob = __shfl_xor(best, o, 64);
    if (oD > D || (oD == D && ob < best)) {
      D = oD;
      best = ob;
    }
  }
  return best;
}

// (I7, I5) of a region from its class sums.
__device__ __forceinline__ double2 rule_values(int d, const double *h, const double (&Sk)[5],
                                               const double *w7, const double *w5) {
  double vol = 1.0;
  for (int j = 0; j < d; ++j) vol *= h[j];
  double r7 = 0.0, r5 = 0.0;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    r7 += w7[k] * Sk[k];
    r5 += w5[k] * Sk[k];
  }
  return make_double2(vol * r7, vol * r5);
}

// One region per W wavefronts; returns (I7, err) in the first thread.
template <int FAM, int W>
__device__ double2 rule_region(const RuleArgs &A, const CSeg &S, long long r, RuleLds &L,
                               double (*part)[5]) {
  const int tid = W == 1 ? threadIdx.x & 63 : threadIdx.x;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  constexpr int NT = 64 * W, LB = W == 1 ? 6 : 8;
  static_assert(NT == 1 << LB, "threads of a region");
  const int d = S.ndim;
  if (tid < d) {
    double cj, hj;
    child_coord(S, r, tid, &cj, &hj);
    L.c[tid] = cj;
    L.h[tid] = hj;
    // both coordinates of every axis at the corners, formed once per region
    // (the values rule_point_f forms per point)
    const double t = A.lam.l5 * hj;
    L.x[2 * tid] = cj + t;
    L.x[2 * tid + 1] = cj - t;
  }
  sync_region<W>();
  double Sk[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  rule_points<FAM>(A.lam, d, tid, NT, LB, L, S.par, S.par + kParamRow, Sk);
#pragma unroll
  for (int k = 0; k < 5; ++k) Sk[k] = wsum(Sk[k]);
  if constexpr (W > 1) {
    if (lane == 0)
#pragma unroll
      for (int k = 0; k < 5; ++k) part[w][k] = Sk[k];
  }
  sync_region<W>();
  if (W > 1 && w != 0) return make_double2(0.0, 0.0);
  if constexpr (W > 1) {
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      Sk[k] = part[0][k];
#pragma unroll
      for (int q = 1; q < W; ++q) Sk[k] += part[q][k];
    }
  }
  const int best = rule_axis(A.lam, d, lane, L.f);
  if (lane == 0) {
    const double2 v = rule_values(d, L.h, Sk, kWeights.w7 + d * 5, kWeights.w5 + d * 5);
    const double err = fabs(v.x - v.y);
    S.regs.I7[r] = v.x;
    S.regs.I5[r] = v.y;
    S.regs.err[r] = err;
    S.regs.axis[r] = best;
    return make_double2(v.x, err);
  }
  return make_double2(0.0, 0.0);
}

// One lane per region, for a single integral of dimension D <= 8: every lane
// takes the rule points in the same order, so the point's class and axes are
// the same across the wavefront (decoded once, in scalar registers) and only
// the region's centre and widths differ.  The point values are the same
// arithmetic as rule_point_f; the class sums are taken in point order.
template <int FAM, int D>
__device__ __forceinline__ double lane_point(const double (&c)[D], const double (&h)[D],
                                             const double *p0, const double *p1,
                                             double phase0, int i, bool ni, int jj, bool nj,
                                             double lam) {
  double acc = Genz<double, FAM>::init(phase0);
#pragma unroll
  for (int j = 0; j < D; ++j) {
    double x = c[j];
    if (j == i || j == jj) {
      const double t = lam * h[j];
      const bool neg = j == i ? ni : nj;
      x = neg ? x - t : x + t;
    }
    acc = Genz<double, FAM>::step(acc, x, p0[j], p1[j]);
  }
  return Genz<double, FAM>::finish(acc, D);
}

// The corners over the axes [J, D) as the leaves of a tree: acc is the running
// value over the axes below J.
template <int FAM, int D, int J>
__device__ __forceinline__ void corner_tree(double acc, const double (&xp)[D],
                                            const double (&xm)[D], const double *p0,
                                            const double *p1, double &s) {
  if constexpr (J == D) {
    s += Genz<double, FAM>::finish(acc, D);
  } else {
    corner_tree<FAM, D, J + 1>(Genz<double, FAM>::step(acc, xp[J], p0[J], p1[J]), xp, xm, p0, p1,
                               s);
    corner_tree<FAM, D, J + 1>(Genz<double, FAM>::step(acc, xm[J], p0[J], p1[J]), xp, xm, p0, p1,
                               s);
  }
}

// Sum over the corners whose signs on the axes below J0 went into acc: a loop
// over the next axes' signs, the last four axes (at most) as an unrolled tree,
// so that a corner costs about two steps and not D.
template <int FAM, int D, int J0>
__device__ __forceinline__ double corner_sum(double acc, const double (&c)[D],
                                             const double (&h)[D], const double *p0,
                                             const double *p1, double l5) {
  constexpr int R = D - J0, IN = R < 4 ? R : 4, M = R - IN;
  double xp[D], xm[D];
#pragma unroll
  for (int j = 0; j < D; ++j) {
    const double t = l5 * h[j];
    xp[j] = c[j] + t;
    xm[j] = c[j] - t;
  }
  double s = 0.0;
  for (unsigned m = 0; m < (1u << M); ++m) {
    double a = acc;
#pragma unroll
    for (int q = 0; q < M; ++q)
      a = Genz<double, FAM>::step(a, ((m >> q) & 1u) ? xm[J0 + q] : xp[J0 + q], p0[J0 + q],
                                  p1[J0 + q]);
    corner_tree<FAM, D, J0 + M>(a, xp, xm, p0, p1, s);
  }
  return s;
}

// All the rule points of one region in one lane (the arithmetic of
// rule_region's points); returns (I7, err).
template <int FAM, int D>
__device__ double2 rule_region_lane(const RuleArgs &A, const CSeg &S, long long r) {
  const long long cap = S.regs.cap;
  double c[D], h[D];
  if (!S.children) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      c[j] = S.regs.c[j * cap + r];
      h[j] = S.regs.h[j * cap + r];
    }
  } else {  // a child: formed from its parent, as child_coord does per axis
    const long long k = r - S.first;
    const long long p = S.parent ? S.parent[k >> 1] : S.pbase + (k >> 1);
    const int ax = S.regs.axis[p];
#pragma unroll
    for (int j = 0; j < D; ++j) {
      c[j] = S.regs.c[j * cap + p];
      h[j] = S.regs.h[j * cap + p];
      if (j == ax) {
        h[j] = h[j] / 2.0;
        c[j] = (k & 1) ? c[j] + h[j] : c[j] - h[j];
      }
      S.regs.c[j * cap + r] = c[j];
      S.regs.h[j * cap + r] = h[j];
    }
    if (S.retire && !(k & 1)) S.regs.err[p] = -1.0;
  }
  const double *p0 = S.par;
  const double *p1 = S.par + kParamRow;
  const double phase0 = p1[0];
  double Sk[5];
  // class 0: the centre
  const double f0 = lane_point<FAM, D>(c, h, p0, p1, phase0, -1, false, -1, false, 0.0);
  Sk[0] = f0;
  // classes 1 and 2: +-lambda on one axis; the fourth differences
  double s1 = 0.0, s2 = 0.0, Dmax = -1.0;
  int best = 0;
  double a2[D];
#pragma unroll
  for (int i = 0; i < D; ++i) {
    const double fp = lane_point<FAM, D>(c, h, p0, p1, phase0, i, false, -1, false, A.lam.l2);
    const double fm = lane_point<FAM, D>(c, h, p0, p1, phase0, i, true, -1, false, A.lam.l2);
    s1 += fp;
    s1 += fm;
    a2[i] = fp + fm - 2.0 * f0;
  }
  const double ratio = (A.lam.l2 * A.lam.l2) / (A.lam.l3 * A.lam.l3);
#pragma unroll
  for (int i = 0; i < D; ++i) {
    const double fp = lane_point<FAM, D>(c, h, p0, p1, phase0, i, false, -1, false, A.lam.l3);
    const double fm = lane_point<FAM, D>(c, h, p0, p1, phase0, i, true, -1, false, A.lam.l3);
    s2 += fp;
    s2 += fm;
    const double a3 = fp + fm - 2.0 * f0;
    const double Dj = fabs(a2[i] - ratio * a3);
    if (Dj > Dmax) {  // strictly greater: the lowest axis wins ties
      Dmax = Dj;
      best = i;
    }
  }
  Sk[1] = s1;
  Sk[2] = s2;
  // class 3: +-lambda4 on two axes i < jj
  double s3 = 0.0;
#pragma unroll
  for (int i = 0; i < D; ++i)
#pragma unroll
    for (int jj = i + 1; jj < D; ++jj)
#pragma unroll
      for (int sg = 0; sg < 4; ++sg)
        s3 += lane_point<FAM, D>(c, h, p0, p1, phase0, i, sg & 1, jj, (sg >> 1) & 1, A.lam.l4);
  Sk[3] = s3;
  // class 4: every corner at +-lambda5
  Sk[4] = corner_sum<FAM, D, 0>(Genz<double, FAM>::init(phase0), c, h, p0, p1, A.lam.l5);
  double vol = 1.0;
#pragma unroll
  for (int j = 0; j < D; ++j) vol *= h[j];
  const double *w7 = kWeights.w7 + D * 5, *w5 = kWeights.w5 + D * 5;
  double r7 = 0.0, r5 = 0.0;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    r7 += w7[k] * Sk[k];
    r5 += w5[k] * Sk[k];
  }
  const double I7 = vol * r7, I5 = vol * r5;
  S.regs.I7[r] = I7;
  S.regs.I5[r] = I5;
  S.regs.err[r] = fabs(I7 - I5);
  S.regs.axis[r] = best;
  return make_double2(I7, fabs(I7 - I5));
}

// The rule points of one region split over the four wavefronts of a block
// (lane l of every wavefront holds region l of the block's 64): wavefront 0
// takes the centre, classes 1 and 2 and the fourth differences; classes 3
// (the pairs of axes, in order, dealt round-robin to wavefronts 1-3) and 4
// (the signs of axes 0 and 1 choose the wavefront) are shared.  Each wavefront's class sums
// go to LDS (sums[w][k][lane]); wavefront 0 adds the four in wavefront order
// and forms I7, I5, err and the split axis.  Returns (I7, err) in
// wavefront 0's lanes of live regions.
template <int FAM, int D>
__device__ double2 rule_region_quad(const RuleArgs &A, const CSeg &S, long long r, bool live,
                                    int w, int lane, double (*sums)[5][64]) {
  const long long cap = S.regs.cap;
  double c[D], h[D];
#pragma unroll
  for (int j = 0; j < D; ++j) c[j] = h[j] = 0.5;  // (a lane past the end computes on these)
  if (live && !S.children) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      c[j] = S.regs.c[j * cap + r];
      h[j] = S.regs.h[j * cap + r];
    }
  } else if (live) {  // a child: formed from its parent, as child_coord does per axis
    const long long k = r - S.first;
    const long long p = S.parent ? S.parent[k >> 1] : S.pbase + (k >> 1);
    const int ax = S.regs.axis[p];
#pragma unroll
    for (int j = 0; j < D; ++j) {
      c[j] = S.regs.c[j * cap + p];
      h[j] = S.regs.h[j * cap + p];
      if (j == ax) {
        h[j] = h[j] / 2.0;
        c[j] = (k & 1) ? c[j] + h[j] : c[j] - h[j];
      }
      if (w == 0) {
        S.regs.c[j * cap + r] = c[j];
        S.regs.h[j * cap + r] = h[j];
      }
    }
    if (w == 0 && S.retire && !(k & 1)) S.regs.err[p] = -1.0;
  }
  const double *p0 = S.par;
  const double *p1 = S.par + kParamRow;
  const double phase0 = p1[0];
  double Sk[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  int best = 0;
  if (w == 0) {
    // class 0: the centre
    const double f0 = lane_point<FAM, D>(c, h, p0, p1, phase0, -1, false, -1, false, 0.0);
    Sk[0] = f0;
    // classes 1 and 2: +-lambda on one axis; the fourth differences
    double s1 = 0.0, s2 = 0.0, Dmax = -1.0;
    double a2[D];
#pragma unroll
    for (int i = 0; i < D; ++i) {
      const double fp = lane_point<FAM, D>(c, h, p0, p1, phase0, i, false, -1, false, A.lam.l2);
      const double fm = lane_point<FAM, D>(c, h, p0, p1, phase0, i, true, -1, false, A.lam.l2);
      s1 += fp;
      s1 += fm;
      a2[i] = fp + fm - 2.0 * f0;
    }
    const double ratio = (A.lam.l2 * A.lam.l2) / (A.lam.l3 * A.lam.l3);
#pragma unroll
    for (int i = 0; i < D; ++i) {
      const double fp = lane_point<FAM, D>(c, h, p0, p1, phase0, i, false, -1, false, A.lam.l3);
      const double fm = lane_point<FAM, D>(c, h, p0, p1, phase0, i, true, -1, false, A.lam.l3);
      s2 += fp;
      s2 += fm;
      const double a3 = fp + fm - 2.0 * f0;
      const double Dj = fabs(a2[i] - ratio * a3);
      if (Dj > Dmax) {  // strictly greater: the lowest axis wins ties
        Dmax = Dj;
        best = i;
      }
    }
    Sk[1] = s1;
    Sk[2] = s2;
  } else {
    // class 3: +-lambda4 on two axes i < jj, pair q to wavefront 1 + q mod 3
    double s3 = 0.0;
    int q = 0;
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
      for (int jj = i + 1; jj < D; ++jj, ++q)
        if (q % 3 == w - 1)
#pragma unroll
          for (int sg = 0; sg < 4; ++sg)
            s3 += lane_point<FAM, D>(c, h, p0, p1, phase0, i, sg & 1, jj, (sg >> 1) & 1, A.lam.l4);
    Sk[3] = s3;
  }
  // class 4: the corners at +-lambda5, the signs of axes 0 and 1 to wavefronts
  {
    double acc = Genz<double, FAM>::init(phase0);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const double t = A.lam.l5 * h[j];
      acc = Genz<double, FAM>::step(acc, ((w >> j) & 1) ? c[j] - t : c[j] + t, p0[j], p1[j]);
    }
    Sk[4] = corner_sum<FAM, D, 2>(acc, c, h, p0, p1, A.lam.l5);
  }
#pragma unroll
  for (int k = 0; k < 5; ++k) sums[w][k][lane] = Sk[k];
  __syncthreads();
  if (w != 0 || !live) return make_double2(0.0, 0.0);
#pragma unroll
  for (int k = 0; k < 5; ++k)
    Sk[k] = ((sums[0][k][lane] + sums[1][k][lane]) + sums[2][k][lane]) + sums[3][k][lane];
  double vol = 1.0;
#pragma unroll
  for (int j = 0; j < D; ++j) vol *= h[j];
  const double *w7 = kWeights.w7 + D * 5, *w5 = kWeights.w5 + D * 5;
  double r7 = 0.0, r5 = 0.0;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    r7 += w7[k] * Sk[k];
    r5 += w5[k] * Sk[k];
  }
  const double I7 = vol * r7, I5 = vol * r5;
  S.regs.I7[r] = I7;
  S.regs.I5[r] = I5;
  S.regs.err[r] = fabs(I7 - I5);
  S.regs.axis[r] = best;
  return make_double2(I7, fabs(I7 - I5));
}

}  // namespace

__global__ void cuhre_root_kernel(CRegions R, int d, int *done) {
  const int j = threadIdx.x;
  if (j < d) {
    R.c[j * R.cap] = 0.5;
    R.h[j * R.cap] = 0.5;
  }
  if (j == 0 && done) *done = 0;
}

// a run's launches do nothing once its stop flag is set
__device__ __forceinline__ bool stopped(const int *done) { return done && *done != 0; }

namespace {

// Sums over a block of up to 1024 threads in a fixed order (a butterfly in
// each wavefront, lane 0's result, then the wavefronts in order); every
// thread gets the sums.
__device__ __forceinline__ double2 block_sum2(double a, double b) {
  __shared__ double s[2][16];
  a = wsum(a);
  b = wsum(b);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();  // an earlier call's readers are done with s
  if ((threadIdx.x & 63) == 0) {
    s[0][w] = a;
    s[1][w] = b;
  }
  __syncthreads();
  double x = 0.0, y = 0.0;
  for (int q = 0; q < nw; ++q) {
    x += s[0][q];
    y += s[1][q];
  }
  return make_double2(x, y);
}

// The stop rule on a step's totals: 0 go on, 1 converged, 2 not finite.
__device__ __forceinline__ int stop_code(double I, double E, const CStop &stop) {
  if (!isfinite(I) || !isfinite(E)) return 2;
  if (stop.neval >= stop.mineval && E <= fmax(stop.epsabs, stop.epsrel * fabs(I))) return 1;
  return 0;
}

// The opening of a step (CRows): true if the run goes on.  Every thread of
// the block must call it.
// (*base: see key_window.)
__device__ __forceinline__ bool open_step(const CRows &R, int *done, int *base = nullptr) {
  if (!R.in) return true;
  double x = 0.0, y = 0.0;
  for (long long i = threadIdx.x; i < R.nin; i += blockDim.x) {
    x += R.in[i];
    y += R.in[R.stride + i];
  }
  const double2 T = block_sum2(x, y);
  const int code = stop_code(T.x, T.y, R.stop);
  const int win = key_window(T.y);
  if (base) *base = win;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (R.window) *R.window = win;
    R.slot[0] = T.x;
    R.slot[1] = T.y;
    __hip_atomic_store((unsigned long long *)(R.slot + 2),
                       ((unsigned long long)R.seq << 8) | (unsigned long long)code,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (code && done) *done = 1;
  }
  return code == 0;
}

// One row of the next state: the block's sums (every thread calls it).
__device__ __forceinline__ void put_row(const CRows &R, double a, double b) {
  if (!R.out) return;
  const double2 t = block_sum2(a, b);
  if (threadIdx.x == 0) {
    R.out[R.out0 + blockIdx.x] = t.x;
    R.out[R.stride + R.out0 + blockIdx.x] = t.y;
  }
}

}  // namespace

// One integral (A.one), dimension D, one lane per region: for launches large
// enough to fill the device with a wavefront per 64 regions.
template <int FAM, int D>
__global__ void __launch_bounds__(256) gm_rule_lane1_kernel(RuleArgs A) {
  if (stopped(A.done) || !open_step(A.rows, A.done)) return;
  const long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  double2 v = make_double2(0.0, 0.0);
  if (g < A.total) v = rule_region_lane<FAM, D>(A, A.one, A.one.first + g);
  put_row(A.rows, v.x, v.y);
}

// One integral (A.one), dimension D: 64 regions per block, one lane of each
// of the block's four wavefronts per region (rule_region_quad).
template <int FAM, int D>
__global__ void __launch_bounds__(256) gm_rule_lane_kernel(RuleArgs A) {
  __shared__ double sums[4][5][64];
  if (stopped(A.done) || !open_step(A.rows, A.done)) return;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const long long g = (long long)blockIdx.x * 64 + lane;
  const double2 v =
      rule_region_quad<FAM, D>(A, A.one, A.one.first + g, g < A.total, w, lane, sums);
  put_row(A.rows, v.x, v.y);
}

// W wavefronts per region, the regions of a launch taken in turn by the grid
// (a launch has at most kWaveRuleBlocks blocks).
template <int W>
__global__ void __launch_bounds__(256) gm_rule_kernel(RuleArgs A) {
  __shared__ RuleLds lds[4 / W];
  __shared__ double part[4][5];
  if (stopped(A.done) || !open_step(A.rows, A.done)) return;
  const int w = W == 1 ? threadIdx.x >> 6 : 0;
  constexpr int RB = 4 / W;  // regions of a block
  double a = 0.0, b = 0.0;
  for (long long g = (long long)blockIdx.x * RB + w; g < A.total;
       g += (long long)gridDim.x * RB) {
    CSeg S;
    long long before = 0;
    if (A.nseg == 1) {
      S = A.one;
    } else {
      int lo = 0, hi = A.nseg - 1;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (A.seg_end[mid] > g)
          hi = mid;
        else
          lo = mid + 1;
      }
      S = A.segs[lo];
      before = lo > 0 ? A.seg_end[lo - 1] : 0;
    }
    const long long r = S.first + (g - before);
    double2 v;
    switch (S.family) {
      case GAUSSIAN: v = rule_region<GAUSSIAN, W>(A, S, r, lds[w], part); break;
      case OSCILLATORY: v = rule_region<OSCILLATORY, W>(A, S, r, lds[w], part); break;
      case PRODUCT_PEAK: v = rule_region<PRODUCT_PEAK, W>(A, S, r, lds[w], part); break;
      case CORNER_PEAK: v = rule_region<CORNER_PEAK, W>(A, S, r, lds[w], part); break;
      default: v = rule_region<C0, W>(A, S, r, lds[w], part); break;
    }
    a += v.x;  // the region's first thread only: the others hold 0
    b += v.y;
    sync_region<W>();  // the region's LDS is reused by the next one
  }
  put_row(A.rows, a, b);
}

// A step opened alone (one block).
__global__ void __launch_bounds__(256) cuhre_decide_kernel(CRows R, int *done) {
  if (stopped(done)) return;
  (void)open_step(R, done);
}

namespace {

// The rule on one region per wavefront, for d = D <= 8: lane l takes the points
// l, l + 64, ..., whose offsets (in half-widths, per axis) it holds in
// registers for every region it takes, so that a point is D multiplications
// and additions and the integrand's own steps, with no decoding and no
// lane-varying branch.  The point values are those of rule_point_f.
template <int FAM, int D>
struct WaveRule {
  static constexpr int NP = (1 << D) + 2 * D * D + 2 * D + 1, PT = (NP + 63) / 64;
  // first points of the classes 0..4, and the end
  static constexpr int kFirst[6] = {0, 1, 1 + 2 * D, 1 + 4 * D, 1 + 4 * D + 2 * D * (D - 1), NP};
  double off[PT][D];
  double p0[D], p1[D];

  __device__ __forceinline__ WaveRule(const RuleLambdas &A, const double *params, int lane) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      p0[j] = uniform(params[j]);
      p1[j] = uniform(params[kParamRow + j]);
    }
#pragma unroll
    for (int k = 0; k < PT; ++k) {
      const int p = lane + 64 * k;
      int i = -1, jj = -1;
      unsigned sgn = 0;
      double lam = 0.0;
      if (p >= kFirst[1] && p < kFirst[3]) {  // classes 1 and 2
        const int q = p - (p < kFirst[2] ? kFirst[1] : kFirst[2]);
        i = q >> 1;
        sgn = q & 1;
        lam = p < kFirst[2] ? A.l2 : A.l3;
      } else if (p >= kFirst[3] && p < kFirst[4]) {
        int q = (p - kFirst[3]) >> 2, row = D - 1;
        sgn = (p - kFirst[3]) & 3;
        i = 0;
        for (; q >= row; --row) {
          q -= row;
          ++i;
        }
        jj = i + 1 + q;
        lam = A.l4;
      } else if (p >= kFirst[4]) {
        sgn = (unsigned)(p - kFirst[4]);
        lam = A.l5;
      }
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const bool corner = p >= kFirst[4];
        const bool on = corner || j == i || j == jj;
        const bool neg = corner ? (sgn >> j) & 1u : j == i ? sgn & 1u : (sgn >> 1) & 1u;
        off[k][j] = !on ? 0.0 : neg ? -lam : lam;
      }
    }
  }

  // The region (c, h): I7 and I5 (in lane 63) and the split axis (in lane 0).
  __device__ __forceinline__ void eval(const RuleLambdas &A, int lane, const double (&c)[D],
                                       const double (&h)[D], const double *w7, const double *w5,
                                       double2 *v, int *axis) const {
    double Sk[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, f0 = 0.0;
#pragma unroll
    for (int k = 0; k < PT; ++k) {
      double acc = Genz<double, FAM>::init(p1[0]);
#pragma unroll
      for (int j = 0; j < D; ++j)
        acc = Genz<double, FAM>::step(acc, c[j] + off[k][j] * h[j], p0[j], p1[j]);
      const double f = Genz<double, FAM>::finish(acc, D);
      if (k == 0) f0 = f;
      const int p = lane + 64 * k;
#pragma unroll
      for (int q = 0; q < 5; ++q)  // (only classes with points among these 64)
        if (kFirst[q] < 64 * k + 64 && kFirst[q + 1] > 64 * k)
          Sk[q] += p >= kFirst[q] && p < kFirst[q + 1] ? f : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) Sk[q] = wave_reduce63_sum(Sk[q]);
    // fourth differences: lane j < D of axis j (its points are the lanes' first)
    const int j = lane & 7;
    const double fc = __shfl(f0, 0, 64);
    const double a2 = __shfl(f0, 1 + 2 * j, 64) + __shfl(f0, 2 + 2 * j, 64) - 2.0 * fc;
    const double a3 =
        __shfl(f0, 1 + 2 * D + 2 * j, 64) + __shfl(f0, 2 + 2 * D + 2 * j, 64) - 2.0 * fc;
    double dm = j < D ? fabs(a2 - (A.l2 * A.l2) / (A.l3 * A.l3) * a3) : -1.0;
    int best = j;
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
      const double od = __shfl_xor(dm, o, 64);
      const int ob = __shfl_xor(best, o, 64);
      if (od > dm || (od == dm && ob < best)) {
        dm = od;
        best = ob;
      }
    }
    *axis = best;
    double vol = 1.0, r7 = 0.0, r5 = 0.0;
#pragma unroll
    for (int q = 0; q < D; ++q) vol *= h[q];
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      r7 += w7[q] * Sk[q];
      r5 += w5[q] * Sk[q];
    }
    *v = make_double2(vol * r7, vol * r5);
  }
};

}  // namespace

// One integral (A.one), d = D <= 8, a wavefront per region: the launches too
// small for a lane per region.  Latency: 64 to 256 regions take 6.8 us at d = 3
// and 7.6 at d = 6, against 9.6 and 12 with the points decoded per region and
// LDS sums.
template <int FAM, int D>
__global__ void __launch_bounds__(256) gm_rule_wave_kernel(RuleArgs A) {
  if (stopped(A.done) || !open_step(A.rows, A.done)) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const long long g = (long long)blockIdx.x * 4 + w;
  double2 t = make_double2(0.0, 0.0);
  if (g < A.total) {
    const CSeg &S = A.one;
    const long long r = S.first + g, cap = S.regs.cap;
    double c[D], h[D];
    if (!S.children) {
#pragma unroll
      for (int j = 0; j < D; ++j) {
        c[j] = S.regs.c[j * cap + r];
        h[j] = S.regs.h[j * cap + r];
      }
    } else {  // a child: formed from its parent, as child_coord does per axis
      const long long p = S.parent ? S.parent[g >> 1] : S.pbase + (g >> 1);
      const int ax = S.regs.axis[p];
#pragma unroll
      for (int j = 0; j < D; ++j) {
        c[j] = S.regs.c[j * cap + p];
        h[j] = S.regs.h[j * cap + p];
      }
#pragma unroll
      for (int j = 0; j < D; ++j)
        if (j == ax) {
          h[j] = h[j] / 2.0;
          c[j] = (g & 1) ? c[j] + h[j] : c[j] - h[j];
        }
#pragma unroll
      for (int j = 0; j < D; ++j)
        if (lane == j) {
          S.regs.c[j * cap + r] = c[j];
          S.regs.h[j * cap + r] = h[j];
        }
      if (S.retire && lane == 0 && !(g & 1)) S.regs.err[p] = -1.0;
    }
    const WaveRule<FAM, D> rule(A.lam, S.par, lane);
    double2 v;
    int axis;
    rule.eval(A.lam, lane, c, h, kWeights.w7 + D * 5, kWeights.w5 + D * 5, &v, &axis);
    if (lane == 0) S.regs.axis[r] = axis;
    if (lane == 63) {
      const double err = fabs(v.x - v.y);
      S.regs.I7[r] = v.x;
      S.regs.I5[r] = v.y;
      S.regs.err[r] = err;
      t = make_double2(v.x, err);
    }
  }
  put_row(A.rows, t.x, t.y);
}

// The first states of a run, while every region splits: one workgroup takes
// the root and A.doublings doublings of the live regions (at most
// kGrowRegions), each generation's regions in LDS and a wavefront per region.
// A launch of its own costs a generation about 10 us, nearly all of it the
// launch and dependent trips to memory that other dies wrote; a generation
// here has none.  Up to 32 regions (six states): 19 us at d = 3, 21 at d = 6.
constexpr int kGrowThreads = 512;

template <int FAM, int D>
__global__ void __launch_bounds__(kGrowThreads) cuhre_grow_kernel(GrowArgs A) {
  constexpr int NW = kGrowThreads / 64;
  __shared__ double sc[2][kGrowRegions][D], sh[2][kGrowRegions][D];
  __shared__ double s7[kGrowRegions], s5[kGrowRegions];
  __shared__ int sax[kGrowRegions];
  __shared__ int s_code;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const WaveRule<FAM, D> rule(A.lam, A.params, lane);
  double w7[5], w5[5];
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    w7[q] = uniform(kWeights.w7[D * 5 + q]);
    w5[q] = uniform(kWeights.w5[D * 5 + q]);
  }
  if (tid < D) sc[0][0][tid] = sh[0][0][tid] = 0.5;
  if (tid == 0) *A.done = 0;
  int n = 1, cur = 0;
  long long base = 0;  // position of the generation's first region
  __syncthreads();
  for (int g = 0;; ++g) {
    for (int r = w; r < n; r += NW) {
      double c[D], h[D];
#pragma unroll
      for (int j = 0; j < D; ++j) {
        c[j] = sc[cur][r][j];
        h[j] = sh[cur][r][j];
      }
      double2 v;
      int axis;
      rule.eval(A.lam, lane, c, h, w7, w5, &v, &axis);
      if (lane == 0) sax[r] = axis;
      if (lane == 63) {
        s7[r] = v.x;
        s5[r] = v.y;
      }
    }
    __syncthreads();
    // the state's totals and outcome
    if (w == 0) {
      const double I = wave_reduce63_sum(lane < n ? s7[lane] : 0.0);
      const double E = wave_reduce63_sum(lane < n ? fabs(s7[lane] - s5[lane]) : 0.0);
      if (lane == 63) {
        int code = 0;
        if (g < A.doublings) {
          CStop stop = A.stop;
          stop.neval = A.np * (2ll * n - 1);
          code = stop_code(I, E, stop);
          if (code || g == A.doublings - 1) {
            A.slot[0] = I;
            A.slot[1] = E;
            __hip_atomic_store((unsigned long long *)(A.slot + 2),
                               ((unsigned long long)g << 8) | (unsigned long long)code,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            if (code) *A.done = 1;
          }
        } else {  // the next launch decides on these
          A.row[0] = I;
          A.row[A.stride] = E;
        }
        s_code = code;
      }
    }
    if (g == A.doublings) break;
    // form the children (not used if the state ends the run)
    for (int e = tid; e < 2 * n * D; e += kGrowThreads) {
      const int k = e / D, j = e % D, p = k >> 1;
      double c = sc[cur][p][j], h = sh[cur][p][j];
      if (j == sax[p]) {
        h = h / 2.0;
        c = (k & 1) ? c + h : c - h;
      }
      sc[cur ^ 1][k][j] = c;
      sh[cur ^ 1][k][j] = h;
    }
    __syncthreads();
    if (s_code) return;
    if (tid < n) A.R.err[base + tid] = -1.0;  // the parents are retired
    base += n;
    n *= 2;
    cur ^= 1;
  }
  for (int e = tid; e < n * D; e += kGrowThreads) {
    const int k = e % n, j = e / n;
    A.R.c[j * A.R.cap + base + k] = sc[cur][k][j];
    A.R.h[j * A.R.cap + base + k] = sh[cur][k][j];
  }
  if (tid < n) {
    A.R.I7[base + tid] = s7[tid];
    A.R.I5[base + tid] = s5[tid];
    A.R.err[base + tid] = fabs(s7[tid] - s5[tid]);
    A.R.axis[base + tid] = sax[tid];
  }
}

// ---------------------------------------------------------------------------
// block-level exclusive scan of per-thread counts (256 threads)

__device__ __forceinline__ long long block_excl_scan(long long v, long long *total) {
  __shared__ long long wtot[kScanBlock / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  long long incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const long long t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  if (lane == 63) wtot[w] = incl;
  __syncthreads();
  long long off = 0, tot = 0;
  for (int q = 0; q < kScanBlock / 64; ++q) {
    if (q < w) off += wtot[q];
    tot += wtot[q];
  }
  __syncthreads();
  *total = tot;
  return off + incl - v;
}

// Whether the region at position i is at or above the threshold (key thr,
// position tpos) in the selection order (key descending, position
// ascending).
__device__ __forceinline__ bool selected(double e, long long i, unsigned long long thr,
                                         long long tpos) {
  const unsigned long long k = key_of(e);
  return k > thr || (k == thr && i <= tpos);
}

constexpr int kTopThreads = 1024;
// Stores up to this many positions have their selected regions counted per tile by
// the gather and the exact ranking, one workgroup over the boundary digit's
// candidates; above, where these can be 10^5 and more, by a launch of its own (4 to
// 9 us).  3 x 10^5 regions a batch at d = 4, oscillatory, to 5 x 10^8 evaluations: 9.88 ms
// with the ranking's count, 9.64 ms with the launch; 10^5 at d = 2, continuous, to 10^8:
// 36.2 and 34.5 ms; below 10^6 regions the two are within 2%.
constexpr long long kCountApart = 1 << 18;
static_assert(kTopThreads == kScanTile, "the gather's passes are the split's tiles");

// Each selected region is retired and its position written to parent[j],
// j its rank in position order: the counts of the tiles before this one
// (summed by every block itself) plus the selected positions before it in
// the tile (the tile's kScanItems chunks of 256 in order, within a chunk the
// wavefronts in order, within a wavefront the lanes below).  With rows, the
// block's sums over the regions that stay live.  Clears the histogram.
__global__ void __launch_bounds__(kScanBlock) split_mark_kernel(double *err, const double *I7,
                                                                long long m,
                                                                const unsigned long long *prefix,
                                                                const long long *krem,
                                                                const long long *bsum,
                                                                long long *parent, long long K,
                                                                unsigned *ghist, CRows rows,
                                                                const int *done) {
  if (stopped(done)) return;
  // (the selection's histogram is clear again for the next one)
  for (int q = blockIdx.x * kScanBlock + threadIdx.x; q < kTopBins; q += gridDim.x * kScanBlock)
    ghist[q] = 0u;
  __shared__ int cnt[kScanItems][kScanBlock / 64];
  const unsigned long long thr = prefix[0];
  const long long tpos = krem[0];
  const long long base = (long long)blockIdx.x * kScanTile;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  long long before = 0;
  for (long long q = threadIdx.x; q < blockIdx.x; q += kScanBlock) before += bsum[q];
  bool f[kScanItems];
  unsigned long long bal[kScanItems];
  double a = 0.0, b = 0.0;
#pragma unroll
  for (int q = 0; q < kScanItems; ++q) {
    const long long i = base + q * kScanBlock + threadIdx.x;
    f[q] = false;
    if (i < m) {
      const double e = err[i];
      f[q] = selected(e, i, thr, tpos);
      if (!f[q] && !retired(e)) {
        a += I7[i];
        b += e;
      }
    }
    bal[q] = __ballot(f[q]);
    if (lane == 0) cnt[q][w] = __popcll(bal[q]);
  }
  long long rank;
  (void)block_excl_scan(before, &rank);  // (also orders cnt's writes before the reads)
  const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
  for (int q = 0; q < kScanItems; ++q) {
    long long pre = 0, all = 0;
#pragma unroll
    for (int v = 0; v < kScanBlock / 64; ++v) {
      if (v < w) pre += cnt[q][v];
      all += cnt[q][v];
    }
    const long long j = rank + pre + __popcll(bal[q] & below);
    if (f[q] && j < K) {  // (exactly K are selected)
      const long long i = base + q * kScanBlock + threadIdx.x;
      parent[j] = i;
      err[i] = -1.0;
    }
    rank += all;
  }
  put_row(rows, a, b);
}

// top-K by a windowed 16-bit first digit ---------------------------------------
//
// The K largest keys, ties to the lower position, in three launches: the
// histogram of the keys' window digits; the digit that holds the K-th key
// (found by every block), the keys and positions of that digit's regions
// gathered, and the count per tile of the regions above it, which are all
// selected; the exact K-th (key, position) among the gathered, whose selected
// ones join the tile counts.  Latency: a 4096-word histogram is cleared, summed
// and scanned in a fraction of what all 65536 digits took (4.4 against 8.2 us a
// launch at d = 3 and 10^4 regions a batch, 6.6 against 11.7 at d = 6 and 10^5),
// and the tile counts need no launch of their own (3.2 us).

__device__ __forceinline__ long long block_excl_scan_1024(long long v, long long *total) {
  __shared__ long long wtot[kTopThreads / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  long long incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const long long t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  if (lane == 63) wtot[w] = incl;
  __syncthreads();
  long long off = 0, tot = 0;
  for (int q = 0; q < kTopThreads / 64; ++q) {
    if (q < w) off += wtot[q];
    tot += wtot[q];
  }
  __syncthreads();
  *total = tot;
  return off + incl - v;
}

// Among nb = 256 * PER digit counts, thread t of 1024 holding the PER
// counts of digits nb - 1 - (PER t + q), q = 0 .. PER - 1 (from the top
// digit down; threads past nb hold none): the digit where the running count
// reaches `need', the need left within it, and its count.
template <int PER>
__device__ __forceinline__ void pick_digit(const long long (&c)[PER], long long need, int nb,
                                           int *dg, long long *left, long long *count) {
  __shared__ int s_dg;
  __shared__ long long s_left, s_cnt;
  const int t = threadIdx.x;
  if (t == 0) {  // (not kept while need <= the total, as it always is)
    s_dg = 0;
    s_left = 1;
    s_cnt = 1;
  }
  long long sum = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) sum += c[q];
  long long tot;
  long long above = block_excl_scan_1024(sum, &tot);
  if (above < need && above + sum >= need) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      if (above + c[q] >= need) {
        s_dg = nb - 1 - (PER * t + q);
        s_left = need - above;
        s_cnt = c[q];
        break;
      }
      above += c[q];
    }
  }
  __syncthreads();
  *dg = s_dg;
  *left = s_left;
  *count = s_cnt;
  __syncthreads();
}

// Opens the step (open), or takes the window from `base' (not negative) or from
// the launch that did (window), and clears the candidate count.
__global__ void __launch_bounds__(kTopThreads) topk_hist_kernel(const double *err, long long m,
                                                                unsigned *ghist,
                                                                unsigned long long *cnt,
                                                                int *window, int base,
                                                                CRows open, int *done) {
  if (stopped(done)) return;
  __shared__ unsigned lh[kTopBins];
  for (int q = threadIdx.x; q < kTopBins; q += kTopThreads) lh[q] = 0u;
  if (open.in) {
    if (!open_step(open, done, &base)) return;
  } else if (base < 0) {
    base = *window;
  } else if (blockIdx.x == 0 && threadIdx.x == 0) {
    *window = base;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) cnt[0] = 0ull;
  __syncthreads();
  constexpr int kKeys = 4;  // loads in flight
  const long long step = (long long)gridDim.x * kTopThreads;
  for (long long i0 = (long long)blockIdx.x * kTopThreads + threadIdx.x; i0 < m;
       i0 += kKeys * step) {
    double e[kKeys];
#pragma unroll
    for (int q = 0; q < kKeys; ++q) e[q] = i0 + q * step < m ? err[i0 + q * step] : -1.0;
#pragma unroll
    for (int q = 0; q < kKeys; ++q) {
      const unsigned long long k = key_of(e[q]);
      if (k) atomicAdd(&lh[window_digit(k, base)], 1u);  // (retired regions are in no digit)
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < kTopBins; q += kTopThreads)
    if (const unsigned c = lh[q]) atomicAdd(&ghist[q], c);
}

// Every block finds the boundary digit; block 0 writes it to prefix[0] and
// the rank wanted within it (from 1) to krem[0].  Then, tile by tile: the keys
// and positions of the digit's regions are gathered (any order, one atomic
// add per tile), and the number of regions above it goes to bsum.
__global__ void __launch_bounds__(kTopThreads) topk_gather_kernel(const double *err, long long m,
                                                                  long long K,
                                                                  const unsigned *ghist,
                                                                  const int *window,
                                                                  unsigned long long *prefix,
                                                                  long long *krem,
                                                                  unsigned long long *ckey,
                                                                  long long *cpos,
                                                                  unsigned long long *cnt,
                                                                  long long *bsum,
                                                                  const int *done) {
  if (stopped(done)) return;
  __shared__ unsigned wc[kTopThreads / 64], wa[kTopThreads / 64];
  __shared__ unsigned long long s_base;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int base = *window;
  int dg;
  long long need, count;
  {
    const uint4 h = ((const uint4 *)ghist)[kTopBins / 4 - 1 - t];  // digits 4095 - 4t down
    const long long c[4] = {(long long)h.w, (long long)h.z, (long long)h.y, (long long)h.x};
    pick_digit<4>(c, K, kTopBins, &dg, &need, &count);
  }
  if (blockIdx.x == 0 && t == 0) {
    prefix[0] = (unsigned long long)dg;
    krem[0] = need;
  }
  for (long long tile = blockIdx.x; tile * kTopThreads < m; tile += gridDim.x) {
    const long long i = tile * kTopThreads + t;
    const unsigned long long k = i < m ? key_of(err[i]) : 0ull;
    const int kd = window_digit(k, base);
    const bool sel = k && kd == dg;
    const unsigned long long bal = __ballot(sel), up = __ballot(k && kd > dg);
    if (lane == 0) {
      wc[w] = (unsigned)__popcll(bal);
      wa[w] = (unsigned)__popcll(up);
    }
    __syncthreads();
    unsigned off = 0, all = 0, above = 0;
    for (int q = 0; q < kTopThreads / 64; ++q) {
      if (q < w) off += wc[q];
      all += wc[q];
      above += wa[q];
    }
    if (t == 0) {
      bsum[tile] = above;
      if (all) s_base = atomicAdd(cnt, (unsigned long long)all);
    }
    __syncthreads();
    if (sel) {
      const unsigned long long o = s_base + off + __popcll(bal & ((1ull << lane) - 1ull));
      ckey[o] = k;
      cpos[o] = i;
    }
    __syncthreads();  // the counts and s_base are rewritten by the next tile
  }
}

// h[d] += 1 for the lanes with sel, in one add where they share d: adds to one
// address follow one another, and so would those of equal keys, of positions that
// differ in other bits, or of one tile's candidates, which the gather wrote together.
__device__ __forceinline__ void count_digit(unsigned *h, int d, bool sel) {
  const unsigned long long any = __ballot(sel);
  if (!any) return;
  const int l = __ffsll((long long)any) - 1;
  const int first = __builtin_amdgcn_readlane(d, l);
  if (__ballot(sel && d != first)) {
    if (sel) atomicAdd(&h[d], 1u);
  } else if ((int)(threadIdx.x & 63) == l) {
    atomicAdd(&h[first], (unsigned)__popcll(any));
  }
}

// One workgroup: among the gathered regions, the one of rank krem[0] (from
// 1) in the order key descending, position ascending: radix passes of 12
// bits over the key's low 48 bits (descending; for the window's digit 0, whose
// keys differ above them too, first two passes of 8), until at most 1024
// candidates share the bits fixed so far, which then rank themselves
// directly; if all bits get fixed first: when the regions with that key
// are not all taken (a tie across the threshold), passes of 8 bits over the
// positions (ascending), else the largest of their positions.  Its key to
// prefix[0], its position to krem[0]; the selected candidates are added to
// the counts of their tiles (of nb; 0: not counted).
__global__ void __launch_bounds__(kTopThreads) topk_exact_kernel(const unsigned long long *ckey,
                                                                 const long long *cpos,
                                                                 const unsigned long long *cnt,
                                                                 const int *window,
                                                                 unsigned long long *prefix,
                                                                 long long *krem,
                                                                 long long *bsum, int nb,
                                                                 const int *done) {
  if (stopped(done)) return;
  __shared__ unsigned h[4096];
  __shared__ unsigned long long s_max;
  const int t = threadIdx.x;
  const unsigned long long dg = prefix[0];
  const long long mc = (long long)cnt[0];
  const int base = *window;
  long long need = krem[0], group = 0;
  // key bits fixed so far: the digit, unless it is the one that smaller keys share
  const bool shared_digit = dg == 0 && base > 0;
  unsigned long long pre = shared_digit ? 0ull : (dg + (unsigned long long)base) << 48;
  unsigned long long mask = shared_digit ? 0ull : 0xFFFFull << 48;
  int dig;
  // up to kExactReg keys per thread, and their positions (below 2^32: a store
  // of 2^32 regions would need over 340 GB), stay in registers
  constexpr int kExactReg = 16;
  constexpr long long kDirect = kTopThreads;  // candidates ranked directly
  const bool inreg = mc <= (long long)kExactReg * kTopThreads;
  unsigned long long kr[kExactReg];
  unsigned pr[kExactReg];
#pragma unroll
  for (int q = 0; q < kExactReg; ++q) {
    const long long i = t + (long long)q * kTopThreads;
    kr[q] = inreg && i < mc ? ckey[i] : 0ull;  // (a live key is not 0)
    pr[q] = inreg && i < mc ? (unsigned)cpos[i] : 0u;
  }
  // f(key, position) over the thread's candidates; more than the registers hold are
  // read again in batches (a load at a time would cost each its way to memory),
  // their positions only if asked for, f getting the candidate's index otherwise
  auto each = [&](auto with_positions, auto f) {
    constexpr bool POS = decltype(with_positions)::value != 0;
    constexpr int kBatch = 4;
    if (inreg) {
#pragma unroll
      for (int q = 0; q < kExactReg; ++q)
        if (kr[q]) f(kr[q], (long long)pr[q]);
    } else {
      for (long long i0 = t; i0 < mc; i0 += kBatch * kTopThreads) {
        unsigned long long kk[kBatch];
        long long pp[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
          const long long i = i0 + (long long)q * kTopThreads;
          kk[q] = i < mc ? ckey[i] : 0ull;
          pp[q] = !POS ? i : i < mc ? cpos[i] : 0;
        }
#pragma unroll
        for (int q = 0; q < kBatch; ++q)
          if (kk[q]) f(kk[q], pp[q]);
      }
    }
  };
  for (int shift = shared_digit ? 56 : 36; shift >= 0; shift -= shift > 48 ? 8 : 12) {
    const unsigned long long bits = shift >= 48 ? 255ull : 4095ull;
    for (int q = t; q < 4096; q += kTopThreads) h[q] = 0u;
    __syncthreads();
    each(Int<0>{}, [&](unsigned long long k, long long) {
      const int d = (int)((k >> shift) & bits);
      const bool sel = (k & mask) == pre;
      if (!inreg)
        count_digit(h, d, sel);
      else if (sel)
        atomicAdd(&h[d], 1u);
    });
    __syncthreads();
    long long c4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) c4[q] = h[4095 - (4 * t + q)];
    pick_digit<4>(c4, need, 4096, &dig, &need, &group);
    pre |= (unsigned long long)dig << shift;
    mask |= bits << shift;
    if (group <= kDirect) break;  // (group is the same in every thread)
  }
  unsigned long long tpos;
  if (group <= kDirect) {
    // few candidates left with the bits fixed so far: each takes its own
    // rank among them directly, (key desc, position asc), and the one of
    // rank need - 1 is the threshold
    __shared__ unsigned long long gk[kDirect];
    __shared__ long long gp[kDirect];
    __shared__ int gcnt;
    __shared__ unsigned long long s_key;
    __shared__ long long s_pos;
    if (t == 0) gcnt = 0;
    __syncthreads();
    each(Int<0>{}, [&](unsigned long long k, long long p) {
      if ((k & mask) == pre) {
        const int o = atomicAdd(&gcnt, 1);
        gk[o] = k;
        gp[o] = inreg ? p : cpos[p];
      }
    });
    __syncthreads();
    const int c = gcnt;
    if (t < c) {
      const unsigned long long mk = gk[t];
      const long long mp = gp[t];
      long long r = 0;
      for (int i = 0; i < c; ++i) r += gk[i] > mk || (gk[i] == mk && gp[i] < mp);
      if (r == need - 1) {
        s_key = mk;
        s_pos = mp;
      }
    }
    __syncthreads();
    pre = s_key;
    tpos = (unsigned long long)s_pos;
  } else if (need == group) {  // every region with the threshold key is taken
    if (t == 0) s_max = 0ull;
    __syncthreads();
    unsigned long long mx = 0ull;
    each(Int<1>{}, [&](unsigned long long k, long long p) {
      if (k == pre) mx = max(mx, (unsigned long long)p);
    });
    atomicMax(&s_max, mx);
    __syncthreads();
    tpos = s_max;
  } else {
    // thread t counts position digit t, which pick_digit sees as
    // digit 255 - t
    unsigned long long ppre = 0ull, pmask = 0xFFFFFFFF00000000ull;
    long long gc;
    for (int shift = 24; shift >= 0; shift -= 8) {
      if (t < 256) h[t] = 0u;
      __syncthreads();
      each(Int<1>{}, [&](unsigned long long k, long long p) {
        count_digit(h, (int)((p >> shift) & 255),
                    k == pre && ((unsigned long long)p & pmask) == ppre);
      });
      __syncthreads();
      const long long c1[1] = {t < 256 ? (long long)h[t] : 0};
      pick_digit<1>(c1, need, 256, &dig, &need, &gc);
      ppre |= (unsigned long long)(255 - dig) << shift;
      pmask |= 255ull << shift;
    }
    tpos = ppre;
  }
  if (t == 0) {
    prefix[0] = pre;
    krem[0] = (long long)tpos;
  }
  // the selected candidates join the gather's counts, summed in LDS (one by one in
  // memory, 16384 candidates of one digit took 60 us)
  if (nb == 0) return;
  __syncthreads();  // (h's last readers)
  for (int q = t; q < nb; q += kTopThreads) h[q] = 0u;
  __syncthreads();
  each(Int<1>{}, [&](unsigned long long k, long long p) {
    count_digit(h, (int)(p / kScanTile), k > pre || (k == pre && p <= (long long)tpos));
  });
  __syncthreads();
  for (int q = t; q < nb; q += kTopThreads)
    if (const unsigned c = h[q]) bsum[q] += c;
}

// The selected regions per tile, for the stores whose exact ranking leaves them out.
__global__ void __launch_bounds__(kScanBlock) sel_count_kernel(const double *err, long long m,
                                                               const unsigned long long *prefix,
                                                               const long long *krem,
                                                               long long *bsum, const int *done) {
  if (stopped(done)) return;
  const unsigned long long thr = prefix[0];
  const long long tpos = krem[0];
  long long n = 0;
#pragma unroll
  for (int q = 0; q < kScanItems; ++q) {
    const long long i = (long long)blockIdx.x * kScanTile + q * kScanBlock + threadIdx.x;
    n += i < m && selected(err[i], i, thr, tpos);
  }
  long long total;
  (void)block_excl_scan(n, &total);
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// totals ---------------------------------------------------------------------

// Sums of I7 and err over the live regions among positions [0, m), per tile
// in a fixed order.
__global__ void __launch_bounds__(kScanBlock) totals_partial_kernel(const double *I7,
                                                                    const double *err,
                                                                    long long m, double *part,
                                                                    const int *done) {
  if (stopped(done)) return;
  const long long base = (long long)blockIdx.x * kScanTile;
  double a = 0.0, b = 0.0;
#pragma unroll
  for (int q = 0; q < kScanItems; ++q) {
    const long long i = base + q * kScanBlock + threadIdx.x;
    if (i < m) {
      const double e = err[i];
      if (!retired(e)) {
        a += I7[i];
        b += e;
      }
    }
  }
  const double2 t = block_sum2(a, b);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = t.x;
    part[gridDim.x + blockIdx.x] = t.y;
  }
}

// One workgroup: the tiles' sums in tile order into out[0..1].
__global__ void __launch_bounds__(kScanBlock) totals_final_kernel(const double *part, long long nb,
                                                                  double *out, const int *done) {
  if (stopped(done)) return;
  double x = 0.0, y = 0.0;
  for (long long i = threadIdx.x; i < nb; i += kScanBlock) {
    x += part[i];
    y += part[nb + i];
  }
  const double2 T = block_sum2(x, y);
  if (threadIdx.x == 0) {
    out[0] = T.x;
    out[1] = T.y;
  }
}

// ---------------------------------------------------------------------------
// launchers

long long scratch_blocks(long long n) { return (n + kScanTile - 1) / kScanTile; }
long long split_rows(long long m) { return scratch_blocks(m); }
long long step_rows(long long cap) {
  return scratch_blocks(cap) + std::max<long long>((cap + 63) / 64, kWaveRuleBlocks);
}

enum RuleSplit { LANE, LANE4, WAVE };  // a lane, a lane of four wavefronts, a wavefront per region

template <int FAM, int D>
static void launch_rule_lane_dd(const RuleArgs &A, unsigned grid, RuleSplit split, hipStream_t s) {
  if constexpr (one_lane_rule(FAM, D))
    if (split == LANE) {
      hipLaunchKernelGGL((gm_rule_lane1_kernel<FAM, D>), dim3(grid), dim3(256), 0, s, A);
      return;
    }
  if (split == WAVE)
    hipLaunchKernelGGL((gm_rule_wave_kernel<FAM, D>), dim3(grid), dim3(256), 0, s, A);
  else
    hipLaunchKernelGGL((gm_rule_lane_kernel<FAM, D>), dim3(grid), dim3(256), 0, s, A);
}

template <int FAM>
static void launch_rule_lane_d(const RuleArgs &A, unsigned grid, RuleSplit split,
                               hipStream_t s) {
  switch (A.one.ndim) {
    case 2: launch_rule_lane_dd<FAM, 2>(A, grid, split, s); break;
    case 3: launch_rule_lane_dd<FAM, 3>(A, grid, split, s); break;
    case 4: launch_rule_lane_dd<FAM, 4>(A, grid, split, s); break;
    case 5: launch_rule_lane_dd<FAM, 5>(A, grid, split, s); break;
    case 6: launch_rule_lane_dd<FAM, 6>(A, grid, split, s); break;
    case 7: launch_rule_lane_dd<FAM, 7>(A, grid, split, s); break;
    default: launch_rule_lane_dd<FAM, 8>(A, grid, split, s); break;
  }
}

template <int FAM>
static void launch_grow_d(const GrowArgs &A, hipStream_t s) {
  const dim3 grid(1), block(kGrowThreads);
  switch (A.d) {
    case 2: hipLaunchKernelGGL((cuhre_grow_kernel<FAM, 2>), grid, block, 0, s, A); break;
    case 3: hipLaunchKernelGGL((cuhre_grow_kernel<FAM, 3>), grid, block, 0, s, A); break;
    case 4: hipLaunchKernelGGL((cuhre_grow_kernel<FAM, 4>), grid, block, 0, s, A); break;
    case 5: hipLaunchKernelGGL((cuhre_grow_kernel<FAM, 5>), grid, block, 0, s, A); break;
    case 6: hipLaunchKernelGGL((cuhre_grow_kernel<FAM, 6>), grid, block, 0, s, A); break;
    case 7: hipLaunchKernelGGL((cuhre_grow_kernel<FAM, 7>), grid, block, 0, s, A); break;
    default: hipLaunchKernelGGL((cuhre_grow_kernel<FAM, 8>), grid, block, 0, s, A); break;
  }
}

hipError_t launch_grow(const GrowArgs &A, int family, hipStream_t s) {
  if (A.d > kGrowMaxDim) return hipErrorInvalidValue;
  switch (family) {
    case GAUSSIAN: launch_grow_d<GAUSSIAN>(A, s); break;
    case OSCILLATORY: launch_grow_d<OSCILLATORY>(A, s); break;
    case PRODUCT_PEAK: launch_grow_d<PRODUCT_PEAK>(A, s); break;
    case CORNER_PEAK: launch_grow_d<CORNER_PEAK>(A, s); break;
    default: launch_grow_d<C0>(A, s); break;
  }
  return hipGetLastError();
}

// One launch in place of two fills and an upload: a run of some 200 us otherwise
// starts with 15 us of them.
constexpr int kSetupPer = 2048;  // parent entries of a block

static __global__ void __launch_bounds__(256) cuhre_setup_kernel(CSetup S) {
  const int tid = threadIdx.x;
  const long long p0 = (long long)blockIdx.x * kSetupPer;
  const long long p1 = min(p0 + kSetupPer, S.nparent);
  for (long long p = p0 + tid; p < p1; p += 256) S.parent[p] = 0;
  if (blockIdx.x > 0) return;
  for (int k = tid; k < kTopBins; k += 256) S.hist[k] = 0;
  if (tid < 2 * kParamRow) S.params_dst[tid] = S.params[tid / kParamRow][tid % kParamRow];
}

hipError_t launch_cuhre_setup(const CSetup &S, hipStream_t s) {
  const long long blocks = S.nparent > kSetupPer ? (S.nparent + kSetupPer - 1) / kSetupPer : 1;
  hipLaunchKernelGGL(cuhre_setup_kernel, dim3((unsigned)blocks), dim3(256), 0, s, S);
  return hipGetLastError();
}

hipError_t launch_root_clear(const CRegions &R, int ndim, int *done, hipStream_t s) {
  hipLaunchKernelGGL(cuhre_root_kernel, dim3(1), dim3(64), 0, s, R, ndim, done);
  return hipGetLastError();
}

// One integral of at most 8 dimensions: a lane per region from
// kOneLaneRuleMinRegions on, where a wavefront per SIMD and more fill the
// device (and one_lane_rule allows it), a lane of each of four wavefronts from kLaneRuleMinRegions, a
// wavefront per region below.  Above 8 dimensions (the registers a lane holds
// grow with d, and the 2^d corners with it) and for launches over several
// integrals, a workgroup or a wavefront per region.
static bool dim_rule(const RuleArgs &A) {
  return A.nseg == 1 && A.one.ndim <= kLaneRuleMaxDim;
}

static RuleSplit rule_split(const RuleArgs &A) {
  if (A.total < kLaneRuleMinRegions) return WAVE;
  return A.total >= kOneLaneRuleMinRegions && one_lane_rule(A.one.family, A.one.ndim) ? LANE
                                                                                      : LANE4;
}

long long rule_blocks(const RuleArgs &A) {
  if (A.total <= 0) return 0;
  if (dim_rule(A)) {
    const long long per[3] = {256, 64, 4};  // regions of a block
    const long long n = per[rule_split(A)];
    return (A.total + n - 1) / n;
  }
  if (A.total <= kBlockRuleRegions) return A.total;
  return std::min<long long>((A.total + 3) / 4, kWaveRuleBlocks);
}

hipError_t launch_rule(const RuleArgs &A, hipStream_t s) {
  const long long grid = rule_blocks(A);
  if (grid <= 0) return hipSuccess;
  if (dim_rule(A)) {
    const RuleSplit q = rule_split(A);
    switch (A.one.family) {
      case GAUSSIAN: launch_rule_lane_d<GAUSSIAN>(A, (unsigned)grid, q, s); break;
      case OSCILLATORY: launch_rule_lane_d<OSCILLATORY>(A, (unsigned)grid, q, s); break;
      case PRODUCT_PEAK: launch_rule_lane_d<PRODUCT_PEAK>(A, (unsigned)grid, q, s); break;
      case CORNER_PEAK: launch_rule_lane_d<CORNER_PEAK>(A, (unsigned)grid, q, s); break;
      default: launch_rule_lane_d<C0>(A, (unsigned)grid, q, s); break;
    }
    return hipGetLastError();
  }
  if (A.total <= kBlockRuleRegions)
    hipLaunchKernelGGL(gm_rule_kernel<4>, dim3((unsigned)grid), dim3(256), 0, s, A);
  else
    hipLaunchKernelGGL(gm_rule_kernel<1>, dim3((unsigned)grid), dim3(256), 0, s, A);
  return hipGetLastError();
}

hipError_t launch_select(const CRegions &R, long long m, long long K, const CScratch &S,
                         hipStream_t s, const CRows *open, const double *E) {
  const int hgrid = (int)std::min<long long>(64, (m + kTopThreads - 1) / kTopThreads);
  const CRows none{};
  hipLaunchKernelGGL(topk_hist_kernel, dim3(hgrid), dim3(kTopThreads), 0, s, R.err, m, S.hist,
                     S.cand_cnt, S.window, E ? key_window(*E) : -1, open ? *open : none, S.done);
  const int ggrid = (int)std::min<long long>(256, (m + kTopThreads - 1) / kTopThreads);
  const bool apart = m > kCountApart;
  hipLaunchKernelGGL(topk_gather_kernel, dim3(ggrid), dim3(kTopThreads), 0, s, R.err, m, K,
                     S.hist, (const int *)S.window, S.prefix, S.krem, S.cand_key, S.cand_pos,
                     S.cand_cnt, S.bsum, (const int *)S.done);
  hipLaunchKernelGGL(topk_exact_kernel, dim3(1), dim3(kTopThreads), 0, s, S.cand_key, S.cand_pos,
                     S.cand_cnt, (const int *)S.window, S.prefix, S.krem, S.bsum,
                     apart ? 0 : (int)scratch_blocks(m), (const int *)S.done);
  if (apart)
    hipLaunchKernelGGL(sel_count_kernel, dim3((unsigned)scratch_blocks(m)), dim3(kScanBlock), 0,
                       s, R.err, m, S.prefix, S.krem, S.bsum, (const int *)S.done);
  return hipGetLastError();
}

hipError_t launch_split(const CRegions &R, long long m, long long K, const CScratch &S,
                        hipStream_t s, const CRows *rows) {
  const long long nb = scratch_blocks(m);
  const CRows none{};
  hipLaunchKernelGGL(split_mark_kernel, dim3((unsigned)nb), dim3(kScanBlock), 0, s, R.err, R.I7,
                     m, S.prefix, S.krem, S.bsum, S.parent, K, S.hist, rows ? *rows : none,
                     (const int *)S.done);
  return hipGetLastError();
}

hipError_t launch_decide(const CRows &rows, int *done, hipStream_t s) {
  hipLaunchKernelGGL(cuhre_decide_kernel, dim3(1), dim3(256), 0, s, rows, done);
  return hipGetLastError();
}

hipError_t launch_totals(const CRegions &R, long long m, const CScratch &S, double *out,
                         hipStream_t s) {
  const long long nb = scratch_blocks(m);
  hipLaunchKernelGGL(totals_partial_kernel, dim3((unsigned)nb), dim3(kScanBlock), 0, s, R.I7,
                     R.err, m, S.tot, (const int *)S.done);
  hipLaunchKernelGGL(totals_final_kernel, dim3(1), dim3(kScanBlock), 0, s, S.tot, nb, out,
                     (const int *)S.done);
  return hipGetLastError();
}

}  // namespace ccuba
