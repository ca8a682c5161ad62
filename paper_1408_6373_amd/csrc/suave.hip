// suave.hip -- Suave's steps on gfx950.
//
// One step of subregion-adaptive Vegas over the regions of one integral:
//   select  the K regions of largest variance (topk: radix select on the
//           variance bits, then a bitonic sort of the K winners by (variance
//           desc, position asc)); one workgroup
//   fluct   per (selected region, dimension, chunk of its stored sample): the
//           two halves' counts, sums and extremes, then the p-th power sums of
//           the deviations from each half's mean (p = flatness), for the L_p
//           fluctuation F_h = (n_h/n) ((1/n_h) sum |v - m_h|^p)^(1/p)
//   split   per selected region: the dimension of least F_0 + F_1, the two
//           children's bounds, their grids (the parent's map restricted to
//           each half along the cut) and the estimates inherited from the
//           parent's sample; one workgroup each
//   sample  DoSample of every child: nnew Philox points through the child's
//           grid (cells staged in LDS), the integrand, v = w V f, the stored
//           (v, side bits) and per-tile sums and v^2 histograms
//   fold    per (child, dimension): the refinement of that dimension of the
//           child's grid; once per child the tile sums in tile order, its own
//           estimate and the inverse-variance combination with the inherited one
//   totals  sums over all regions, the stop rule and, at the end, the chi^2
//           probability; one workgroup
// Steps are queued ahead of their totals: select and fluct change no region,
// so the host learns a step's outcome while the next step's run.
#include "engine.h"
#include "genz.h"
#include "philox.h"
#include "refine.h"
#include "suave.h"
#include "wave.h"

namespace ccuba {

namespace {

// sum of one double per thread over the block, in a fixed order; every thread
// gets the result (red: blockDim/64 doubles of LDS)
__device__ double block_sum(double v, double *red) {
  v = wave_sum(v);
  const int nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  for (int q = 0; q < nw; ++q) s += red[q];
  return s;
}

// exclusive prefix sum of one int per thread over the block (block of 1024)
__device__ int block_scan_excl(int v, int *red, int *total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  __syncthreads();
  if (lane == 63) red[w] = incl;
  __syncthreads();
  int before = 0, all = 0;
  for (int q = 0; q < nw; ++q) {
    if (q < w) before += red[q];
    all += red[q];
  }
  *total = all;
  return before + incl - v;
}

__device__ __forceinline__ unsigned long long var_key(double x) {
  return (unsigned long long)__double_as_longlong(x);  // variances are >= 0
}

}  // namespace

__global__ void __launch_bounds__(256) suave_root_kernel(SuaveArgs A) {
  const int d = A.d, N = A.N;
  for (int e = threadIdx.x; e < d * (N + 1); e += blockDim.x)
    A.R.grid[e] = (double)(e % (N + 1)) / N;
  if (threadIdx.x < d) {
    A.R.lo[threadIdx.x] = 0.0;
    A.R.hi[threadIdx.x] = 1.0;
  }
  if (threadIdx.x == 0) {
    A.R.inh_I[0] = 0.0;
    A.R.inh_var[0] = 0.0;
    A.chpos[0] = 0;
    A.chser[0] = 0;
  }
}

constexpr int kKeyRegs = 8;     // keys a thread of the selection holds in registers
constexpr int kTopGroup = 64;   // boundary keys ranked directly

// The K largest of R non-negative keys, ties to the lower position, in that
// order (the regions of largest variance here, of largest spread in the
// Divonne partition): 8-bit digits from the highest bit in which any two keys
// differ, until at most 64 keys share the boundary digits (they rank
// themselves) or all that do are taken; then a bitonic sort of the K winners.
// One workgroup: latency.  Up to 8192 keys stay in registers over the passes.
// 1024 of up to 8192 keys: 14.7 us on average, 17.6 with every step of the sort
// through LDS, 24.3 with eight passes that read the keys from memory as well; 64
// of up to 1000: 9.5, 10.4 and 14.8.
__global__ void __launch_bounds__(1024) topk_kernel(const double *key, int R, int K, int *sel) {
  __shared__ unsigned hist[2][256];
  __shared__ unsigned long long wmax[16], wmin[16];
  __shared__ unsigned long long s_prefix;
  __shared__ int s_krem, s_group, s_take, s_ng;
  __shared__ int red[16];
  __shared__ unsigned long long gkey[kTopGroup];
  __shared__ int gpos[kTopGroup];
  __shared__ unsigned long long skey[kSuaveMaxSplit];
  __shared__ int spos[kSuaveMaxSplit];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const bool inreg = R <= kKeyRegs * 1024;
  unsigned long long kr[kKeyRegs];
#pragma unroll
  for (int q = 0; q < kKeyRegs; ++q)
    kr[q] = inreg && tid + 1024 * q < R ? var_key(key[tid + 1024 * q]) : 0;
  // f(key, position) over the thread's keys
  auto each = [&](auto f) {
    if (inreg) {
#pragma unroll
      for (int q = 0; q < kKeyRegs; ++q)
        if (tid + 1024 * q < R) f(kr[q], tid + 1024 * q);
    } else {
      for (int i0 = tid; i0 < R; i0 += 1024 * kKeyRegs) {
        unsigned long long kk[kKeyRegs];
#pragma unroll
        for (int q = 0; q < kKeyRegs; ++q)
          kk[q] = i0 + 1024 * q < R ? var_key(key[i0 + 1024 * q]) : 0;
#pragma unroll
        for (int q = 0; q < kKeyRegs; ++q)
          if (i0 + 1024 * q < R) f(kk[q], i0 + 1024 * q);
      }
    }
  };
  // the bits that all keys share need no pass
  unsigned long long mx = 0, mn = ~0ull;
  each([&](unsigned long long k, int) {
    mx = max(mx, k);
    mn = min(mn, k);
  });
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    mx = max(mx, (unsigned long long)__shfl_xor((long long)mx, o, 64));
    mn = min(mn, (unsigned long long)__shfl_xor((long long)mn, o, 64));
  }
  if (lane == 0) {
    wmax[w] = mx;
    wmin[w] = mn;
  }
  if (tid < 512) hist[tid >> 8][tid & 255] = 0;
  if (tid == 0) {
    s_take = 0;
    s_ng = 0;
  }
  __syncthreads();
  for (int q = 0; q < 16; ++q) {
    mx = max(mx, wmax[q]);
    mn = min(mn, wmin[q]);
  }
  const int top = mx == mn ? 0 : 64 - __clzll((long long)(mx ^ mn));  // bits that differ
  int shift = max(0, (top + 7) / 8 * 8);
  unsigned long long mask = shift >= 64 ? 0 : ~0ull << shift, pre = mx & mask;
  int krem = K, group = R, par = 0;
  while (shift > 0 && group > kTopGroup && group != krem) {
    shift -= 8;
    each([&](unsigned long long k, int) {
      if ((k & mask) == pre) atomicAdd(&hist[par][(k >> shift) & 255], 1u);
    });
    __syncthreads();
    if (tid < 64) {  // one wavefront: lane l owns digits 4l .. 4l+3
      unsigned hh[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) hh[q] = hist[par][4 * lane + q];
      const unsigned mine = hh[0] + hh[1] + hh[2] + hh[3];
      // count of keys with a larger digit: the lanes above, inclusive scan downwards
      unsigned above = mine;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const unsigned t = __shfl_down(above, o, 64);
        if (lane + o < 64) above += t;
      }
      unsigned cum = above - mine;
      for (int q = 3; q >= 0; --q) {
        if (cum < (unsigned)krem && (unsigned)krem <= cum + hh[q]) {
          s_krem = krem - (int)cum;
          s_group = (int)hh[q];
          s_prefix = pre | ((unsigned long long)(4 * lane + q) << shift);
        }
        cum += hh[q];
      }
    } else if (tid >= 256 && tid < 512) {
      hist[par ^ 1][tid - 256] = 0;  // (read last before the barrier above)
    }
    __syncthreads();
    pre = s_prefix;
    krem = s_krem;
    group = s_group;
    mask |= 255ull << shift;
    par ^= 1;
  }
  // above the boundary digits: all taken; within them: krem of the group
  const bool all = group == krem;
  each([&](unsigned long long k, int i) {
    const unsigned long long b = k & mask;
    if (b > pre || (all && b == pre)) {
      const int o = atomicAdd(&s_take, 1);
      skey[o] = k;
      spos[o] = i;
    } else if (b == pre && group <= kTopGroup) {
      const int o = atomicAdd(&s_ng, 1);
      gkey[o] = k;
      gpos[o] = i;
    }
  });
  int P = 1;
  while (P < K) P <<= 1;
  for (int i = K + tid; i < P; i += 1024) {
    skey[i] = 0;
    spos[i] = 0x7fffffff;
  }
  __syncthreads();
  if (!all && group <= kTopGroup) {
    if (tid < group) {
      const unsigned long long mk = gkey[tid];
      const int mp = gpos[tid];
      int r = 0;
      for (int q = 0; q < group; ++q) r += gkey[q] > mk || (gkey[q] == mk && gpos[q] < mp);
      if (r < krem) {
        skey[K - krem + r] = mk;
        spos[K - krem + r] = mp;
      }
    }
  } else if (!all) {  // every bit is fixed: equal keys, the lowest positions first
    int base = 0;
    for (int i0 = 0; i0 < R && base < krem; i0 += 1024) {
      const int i = i0 + tid;
      const unsigned long long k = i < R ? var_key(key[i]) : 0;
      const int eq = i < R && (k & mask) == pre;
      int tot;
      const int o = base + block_scan_excl(eq, red, &tot);
      if (eq && o < krem) {
        skey[K - krem + o] = k;
        spos[K - krem + o] = i;
      }
      base += tot;
    }
  }
  __syncthreads();
  // bitonic sort, an element a thread: larger key first, then lower position.
  // Partners of the same wavefront exchange by shuffles; only strides from 64 on go
  // through LDS and its barriers (10 of the 55 steps for 1024 elements).
  unsigned long long mk = tid < P ? skey[tid] : 0;
  int mp = tid < P ? spos[tid] : 0;
  for (int size = 2; size <= P; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      unsigned long long ok;
      int op;
      if (stride >= 64) {
        __syncthreads();
        if (tid < P) {
          skey[tid] = mk;
          spos[tid] = mp;
        }
        __syncthreads();
        if (tid >= P) continue;
        ok = skey[tid ^ stride];
        op = spos[tid ^ stride];
      } else {
        if ((tid & ~63) >= P) continue;  // (whole wavefronts)
        ok = (unsigned long long)__shfl_xor((long long)mk, stride, 64);
        op = __shfl_xor(mp, stride, 64);
      }
      const bool first = mk > ok || (mk == ok && mp < op);
      if (first != (((tid & stride) == 0) == ((tid & size) == 0))) {
        mk = ok;
        mp = op;
      }
    }
  if (tid < K) sel[tid] = mp;
}

// Split statistics in two passes over each selected region's sample, both
// spread over chunks of A.chunk points (grid: chunk x region):
//   pass 1, per (dimension, half): count, S1 = sum v, S2 = sum v^2, min v and
//           max v; the largest deviation from the half's mean m_h is then
//           exactly M_h = max(vmax - m_h, m_h - vmin);
//   pass 2, per (dimension, half): sum (|v - m_h| / M_h)^p.
// Chunk partials are reduced in a fixed order wherever they are needed.
//
// Both passes are bound by VALU issue (14 and 17 instructions per point and
// dimension at p = 25).  A thread keeps the partial sums of kFlDims dimensions
// in registers and reads its points from memory, so no point passes through
// LDS; a workgroup's dimension groups read the same points at about the same
// time.  The half of a point enters as a bit mask: factors 0.0 and 1.0 of
// fused multiply-adds, and quiet NaNs, which minimum and maximum pass over.
// Every factor's partner is finite, or a point would reach the other half as 0.0
// times infinity: a square that overflows enters as the largest finite number, and
// a deviation below the smallest normal, whose reciprocal overflows, is scaled by
// the smallest normal instead (F_h is the same for every scale).
// 64 regions of 2^17 points, d = 8, p = 25: 30 and 45 us a launch, against 59 and
// 66 (and 7 for a reduction launch between them) with the chunks staged in LDS
// and a thread per (dimension, point).
constexpr int kP1 = 9;         // per (chunk, dimension): cnt1, S1_0, S2_0, S1_1, S2_1, min0, max0, min1, max1
constexpr int kHs = 10;        // per (region, dimension): cnt, S1, S2, m, M of each half
constexpr int kFlDims = 4;     // dimensions of a thread
constexpr int kFlThreads = 128;  // threads that share a dimension group
constexpr int kFlGroups = kMaxDim / kFlDims;
constexpr int kFlItems = kFlDims * kP1;  // pass-1 values of a dimension group

namespace {

// a double made of a high word (0.0 and 1.0 have a zero low word)
__device__ __forceinline__ double hi_double(uint32_t hi) {
  return __longlong_as_double((long long)((unsigned long long)hi << 32));
}

// v_min_f64 / v_max_f64 as they are: of a number and a quiet NaN, the number
__device__ __forceinline__ double min_num(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double max_num(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

__device__ __forceinline__ double p1_merge(int q, double x, double y) {
  return (q == 5 || q == 7) ? fmin(x, y) : (q == 6 || q == 8) ? fmax(x, y) : x + y;
}
__device__ __forceinline__ double p1_identity(int q) {
  return (q == 5 || q == 7) ? INFINITY : (q == 6 || q == 8) ? -INFINITY : 0.0;
}

// U points (stride kFlThreads) of a thread at a time, f(x, bits of its
// dimension group) for each of its points
template <int U, typename F>
__device__ __forceinline__ void each_points(const double *v, const uint16_t *sd, int cnt, int g,
                                            F f) {
  int i = threadIdx.x & (kFlThreads - 1);
  for (; i + (U - 1) * kFlThreads < cnt; i += U * kFlThreads) {
    double x[U];
    uint32_t b[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      x[q] = v[i + q * kFlThreads];
      b[q] = (uint32_t)sd[i + q * kFlThreads] >> (kFlDims * g);
    }
    f(x, b);
  }
  for (; i < cnt; i += kFlThreads) {  // (x and bits of a missing point: see the callers)
    double x[U];
    uint32_t b[U];
    x[0] = v[i];
    b[0] = (uint32_t)sd[i] >> (kFlDims * g);
    f(x, b, 1);
  }
}

// -1 if bit q of b is set, else 0
__device__ __forceinline__ uint32_t bit_mask(uint32_t b, int q) {
  return (uint32_t)((int)(b << (31 - q)) >> 31);
}

}  // namespace

// Pass 1 over one chunk: grid (chunk, selected region).
__global__ void __launch_bounds__(kFlThreads *kFlGroups) suave_fluct1_kernel(SuaveArgs A) {
  __shared__ double red[kFlGroups][2][kFlItems];
  const int ch = blockIdx.x, s = blockIdx.y, tid = threadIdx.x, d = A.d;
  const int g = __builtin_amdgcn_readfirstlane(tid / kFlThreads), t = tid % kFlThreads;
  const long long i0 = (long long)ch * A.chunk;
  const int cnt = (int)min((long long)A.chunk, A.nnew - i0);
  const size_t at = (size_t)A.sel[s] * A.nnew + i0;
  double s1l[kFlDims], s2l[kFlDims], s1u[kFlDims], s2u[kFlDims];
  double mnl[kFlDims], mxl[kFlDims], mnu[kFlDims], mxu[kFlDims];
  uint32_t cu[kFlDims];
#pragma unroll
  for (int q = 0; q < kFlDims; ++q) {
    s1l[q] = s2l[q] = s1u[q] = s2u[q] = 0.0;
    mnl[q] = mnu[q] = INFINITY;
    mxl[q] = mxu[q] = -INFINITY;
    cu[q] = 0;
  }
  constexpr int U = 4;
  each_points<U>(A.R.v + at, A.R.side + at, cnt, g,
                 [&](const double (&x)[U], const uint32_t (&b)[U], int m = U) {
#pragma unroll
    for (int p = 0; p < U; ++p) {
      if (p >= m) break;
      const double xx = min_num(x[p] * x[p], 0x1.fffffffffffffp1023);
      const unsigned long long xb = (unsigned long long)__double_as_longlong(x[p]);
      const uint32_t xh = (uint32_t)(xb >> 32);
#pragma unroll
      for (int q = 0; q < kFlDims; ++q) {
        const uint32_t up = bit_mask(b[p], q);
        const double fu = hi_double(up & 0x3FF00000u), fl = hi_double(~up & 0x3FF00000u);
        s1l[q] = fma(fl, x[p], s1l[q]);
        s2l[q] = fma(fl, xx, s2l[q]);
        s1u[q] = fma(fu, x[p], s1u[q]);
        s2u[q] = fma(fu, xx, s2u[q]);
        cu[q] -= up;
        const unsigned long long lo = xb & 0xFFFFFFFFull;
        const double xl = __longlong_as_double(
            (long long)(((unsigned long long)(xh | (up & 0x7FF80000u)) << 32) | lo));
        const double xu = __longlong_as_double(
            (long long)(((unsigned long long)(xh | (~up & 0x7FF80000u)) << 32) | lo));
        mnl[q] = min_num(mnl[q], xl);
        mxl[q] = max_num(mxl[q], xl);
        mnu[q] = min_num(mnu[q], xu);
        mxu[q] = max_num(mxu[q], xu);
      }
    }
  });
  auto mn = [](double a, double b) { return min_num(a, b); };
  auto mx = [](double a, double b) { return max_num(a, b); };
  const int w = (tid >> 6) & 1;
#pragma unroll
  for (int q = 0; q < kFlDims; ++q) {
    const double r[kP1] = {wave_reduce63_sum((double)cu[q]), wave_reduce63_sum(s1l[q]),
                           wave_reduce63_sum(s2l[q]),        wave_reduce63_sum(s1u[q]),
                           wave_reduce63_sum(s2u[q]),        wave_reduce63(mnl[q], INFINITY, mn),
                           wave_reduce63(mxl[q], -INFINITY, mx),
                           wave_reduce63(mnu[q], INFINITY, mn),
                           wave_reduce63(mxu[q], -INFINITY, mx)};
    if ((tid & 63) == 63)
#pragma unroll
      for (int k = 0; k < kP1; ++k) red[g][w][q * kP1 + k] = r[k];
  }
  __syncthreads();
  const int j = kFlDims * g + t / kP1;
  if (t < kFlItems && j < d)
    A.fl1[(((size_t)s * A.nchunks + ch) * d + j) * kP1 + t % kP1] =
        p1_merge(t % kP1, red[g][0][t], red[g][1][t]);
}

// Pass 2 over one chunk: grid (chunk, selected region).  Each workgroup first
// reduces pass 1 over the chunks (kFlSegs threads a value); chunk 0's writes
// the halves' statistics for the split.
constexpr int kFlSegs = kFlThreads / kFlItems;

__global__ void __launch_bounds__(kFlThreads *kFlGroups) suave_fluct2_kernel(SuaveArgs A) {
  __shared__ double part[kFlGroups][kFlSegs][kFlItems];
  __shared__ double sm[kMaxDim][2], sinv[kMaxDim][2];
  __shared__ double red[kFlGroups][2][2 * kFlDims];
  const int ch = blockIdx.x, s = blockIdx.y, tid = threadIdx.x, d = A.d;
  const int g = __builtin_amdgcn_readfirstlane(tid / kFlThreads), t = tid % kFlThreads;
  {
    const int seg = t / kFlItems, item = t - seg * kFlItems;
    const int j = kFlDims * g + item / kP1, q = item % kP1;
    if (seg < kFlSegs && j < d) {
      double a = p1_identity(q);
      const double *r = A.fl1 + ((size_t)s * A.nchunks * d + j) * kP1 + q;
#pragma unroll 8
      for (int c = seg; c < A.nchunks; c += kFlSegs) a = p1_merge(q, a, r[(size_t)c * d * kP1]);
      part[g][seg][item] = a;
    }
  }
  __syncthreads();
  if (t < kFlDims && kFlDims * g + t < d) {
    const int j = kFlDims * g + t;
    double x[kP1];
#pragma unroll
    for (int q = 0; q < kP1; ++q) {
      x[q] = part[g][0][t * kP1 + q];
#pragma unroll
      for (int k = 1; k < kFlSegs; ++k) x[q] = p1_merge(q, x[q], part[g][k][t * kP1 + q]);
    }
    const double cnt[2] = {(double)A.nnew - x[0], x[0]};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const double S1 = x[1 + 2 * k], mn = x[5 + 2 * k], mx = x[6 + 2 * k];
      const double m = cnt[k] > 0.0 ? S1 / cnt[k] : 0.0;
      double M = cnt[k] > 0.0 ? fmax(mx - m, m - mn) : 0.0;
      if (M > 0.0) M = fmax(M, 0x1p-1022);
      sm[j][k] = m;
      sinv[j][k] = M > 0.0 ? 1.0 / M : 0.0;
      if (ch == 0) {
        double *o = A.hs + ((size_t)s * d + j) * kHs + 5 * k;
        o[0] = cnt[k];
        o[1] = S1;
        o[2] = x[2 + 2 * k];
        o[3] = m;
        o[4] = M;
      }
    }
  }
  __syncthreads();
  double m0[kFlDims], m1[kFlDims], i0v[kFlDims], i1v[kFlDims], ql[kFlDims], qu[kFlDims];
#pragma unroll
  for (int q = 0; q < kFlDims; ++q) {
    const int j = kFlDims * g + q;
    m0[q] = j < d ? sm[j][0] : 0.0;
    m1[q] = j < d ? sm[j][1] : 0.0;
    i0v[q] = j < d ? sinv[j][0] : 0.0;
    i1v[q] = j < d ? sinv[j][1] : 0.0;
    ql[q] = qu[q] = 0.0;
  }
  const double p = A.flatness;
  const int ip = A.ipow;
  const long long i0 = (long long)ch * A.chunk;
  const int cnt = (int)min((long long)A.chunk, A.nnew - i0);
  const size_t at = (size_t)A.sel[s] * A.nnew + i0;
  constexpr int U = 4;
  each_points<U>(A.R.v + at, A.R.side + at, cnt, g,
                 [&](const double (&x)[U], const uint32_t (&b)[U], int m = U) {
    double r[U][kFlDims], y[U][kFlDims];
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (k < m)
#pragma unroll
        for (int q = 0; q < kFlDims; ++q) {
          const bool up = (b[k] >> q) & 1u;
          r[k][q] = fabs(x[k] - (up ? m1[q] : m0[q])) * (up ? i1v[q] : i0v[q]);
        }
      else
#pragma unroll
        for (int q = 0; q < kFlDims; ++q) r[k][q] = 0.0;
    if (ip > 0) {  // r^p by squaring, from the lowest bit of p; every value together
      int e = ip;
      for (; !(e & 1); e >>= 1)
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
          for (int q = 0; q < kFlDims; ++q) r[k][q] *= r[k][q];
#pragma unroll
      for (int k = 0; k < U; ++k)
#pragma unroll
        for (int q = 0; q < kFlDims; ++q) y[k][q] = r[k][q];
      for (e >>= 1; e; e >>= 1) {
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
          for (int q = 0; q < kFlDims; ++q) r[k][q] *= r[k][q];
        if (e & 1)
#pragma unroll
          for (int k = 0; k < U; ++k)
#pragma unroll
            for (int q = 0; q < kFlDims; ++q) y[k][q] *= r[k][q];
      }
    } else {
#pragma unroll
      for (int k = 0; k < U; ++k)
#pragma unroll
        for (int q = 0; q < kFlDims; ++q)
          y[k][q] = r[k][q] > 0.0 ? exp2(p * log2(r[k][q])) : 0.0;
    }
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (k < m)
#pragma unroll
        for (int q = 0; q < kFlDims; ++q) {
          const uint32_t up = bit_mask(b[k], q);
          ql[q] = fma(hi_double(~up & 0x3FF00000u), y[k][q], ql[q]);
          qu[q] = fma(hi_double(up & 0x3FF00000u), y[k][q], qu[q]);
        }
  });
  const int w = (tid >> 6) & 1;
#pragma unroll
  for (int q = 0; q < kFlDims; ++q) {
    const double a = wave_reduce63_sum(ql[q]), c = wave_reduce63_sum(qu[q]);
    if ((tid & 63) == 63) {
      red[g][w][2 * q] = a;
      red[g][w][2 * q + 1] = c;
    }
  }
  __syncthreads();
  const int j = kFlDims * g + (t >> 1);
  if (t < 2 * kFlDims && j < d)
    A.fl2[(((size_t)s * A.nchunks + ch) * d + j) * 2 + (t & 1)] = red[g][0][t] + red[g][1][t];
}

namespace {

// the parent's map along one dimension, X(y), piecewise linear through (k/N, E_k)
__device__ __forceinline__ double map_at(const double *E, int N, double y) {
  const double z = y * N;
  int k = (int)floor(z);
  k = min(max(k, 0), N - 1);
  return fma(z - k, E[k + 1] - E[k], E[k]);
}

// running maximum over e[0..n) by one wavefront (lanes own contiguous runs)
__device__ void wave_prefix_max(double *e, int n, int lane) {
  const int per = (n + 63) >> 6;
  const int k0 = min(lane * per, n), k1 = min(k0 + per, n);
  double run = -INFINITY;
  for (int k = k0; k < k1; ++k) run = fmax(run, e[k]);
  double incl = run;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double t = __shfl_up(incl, o, 64);
    if (lane >= o) incl = fmax(incl, t);
  }
  double acc = __shfl_up(incl, 1, 64);
  if (lane == 0) acc = -INFINITY;
  for (int k = k0; k < k1; ++k) {
    acc = fmax(acc, e[k]);
    e[k] = acc;
  }
}

}  // namespace

// Per selected region: the cut and the two children.
__global__ void __launch_bounds__(256) suave_split_kernel(SuaveArgs A, int R, long long Q) {
  __shared__ double sE[kMaxBins + 1];
  __shared__ double sOut[2][kMaxBins + 1];
  __shared__ int s_cut, s_ks;
  const int s = blockIdx.x, tid = threadIdx.x;
  const int d = A.d, N = A.N, row = N + 1;
  const int pos = A.sel[s], up = R + s;
  constexpr int kItems = 2 * kMaxDim, kSegs = 256 / kItems;
  __shared__ double s_part[kSegs][kItems], s_term[kItems], s_score[kMaxDim], s_S[kMaxDim][4];
  {  // pass 2 over the chunks: item 2j + k in kSegs interleaved runs
    const int seg = tid / kItems, item = tid % kItems;
    double q = 0.0;
    if (item < 2 * d) {
      const double *r = A.fl2 + (size_t)s * A.nchunks * d * 2 + item;
#pragma unroll 8
      for (int ch = seg; ch < A.nchunks; ch += kSegs) q += r[(size_t)ch * d * 2];
    }
    s_part[seg][item] = q;
  }
  __syncthreads();
  if (tid < 2 * d) {  // one half's term of a cut along dimension tid / 2
    const double *h = A.hs + ((size_t)s * d + (tid >> 1)) * kHs + 5 * (tid & 1);
    const double nd = (double)A.nnew, p = A.flatness;
    double q = s_part[0][tid];
    for (int k = 1; k < kSegs; ++k) q += s_part[k][tid];
    const double cnt = h[0], M = h[4];
    s_term[tid] = cnt > 0.0 && M > 0.0 ? (cnt / nd) * M * pow(q / cnt, 1.0 / p) : 0.0;
    s_S[tid >> 1][2 * (tid & 1)] = h[1];
    s_S[tid >> 1][2 * (tid & 1) + 1] = h[2];
  }
  __syncthreads();
  if (tid < d) s_score[tid] = s_term[2 * tid] + s_term[2 * tid + 1];
  __syncthreads();
  if (tid == 0) {
    int best = 0;
    double b = s_score[0];
    for (int c = 1; c < d; ++c)
      if (s_score[c] < b) {
        b = s_score[c];
        best = c;
      }
    s_cut = best;
    A.cut[Q + s] = best;
  }
  __syncthreads();
  const int c = s_cut;
  double *Gp = A.R.grid + (size_t)pos * d * row;
  double *Gu = A.R.grid + (size_t)up * d * row;
  for (int e = tid; e < d * row; e += 256) Gu[e] = Gp[e];
  for (int e = tid; e <= N; e += 256) sE[e] = Gp[c * row + e];
  if (tid < d) {
    A.R.lo[(size_t)up * d + tid] = A.R.lo[(size_t)pos * d + tid];
    A.R.hi[(size_t)up * d + tid] = A.R.hi[(size_t)pos * d + tid];
  }
  __syncthreads();
  if (tid == 0) {
    const double mid = 0.5 * (A.R.lo[(size_t)pos * d + c] + A.R.hi[(size_t)pos * d + c]);
    A.R.hi[(size_t)pos * d + c] = mid;
    A.R.lo[(size_t)up * d + c] = mid;
    const double n = (double)A.nnew;
    for (int h = 0; h < 2; ++h) {
      const double I = s_S[c][2 * h] / n;
      const double var = fmax(0.0, s_S[c][2 * h + 1] / n - I * I) / (n - 1.0);
      const int p = h == 0 ? pos : up;
      A.R.inh_I[p] = var > 0.0 ? I : 0.0;
      A.R.inh_var[p] = var > 0.0 ? var : 0.0;
    }
    A.chpos[2 * s] = pos;
    A.chpos[2 * s + 1] = up;
    A.chser[2 * s] = (int)(2 * (Q + s) + 1);
    A.chser[2 * s + 1] = (int)(2 * (Q + s) + 2);
  }
  // the bin holding 1/2: the first k with E_k+1 > 1/2 (at most N - 1)
  if (tid == 0) s_ks = N - 1;
  __syncthreads();
  for (int k = tid; k < N; k += 256)
    if (sE[k + 1] > 0.5) atomicMin(&s_ks, k);
  __syncthreads();
  const int ks = s_ks;
  const double ystar = (ks + (0.5 - sE[ks]) / (sE[ks + 1] - sE[ks])) / N;
  for (int k = tid; k <= N; k += 256) {
    const double t = (double)k / N;
    sOut[0][k] = 2.0 * map_at(sE, N, ystar * t);
    sOut[1][k] = 2.0 * map_at(sE, N, fma(1.0 - ystar, t, ystar)) - 1.0;
  }
  __syncthreads();
  if (tid == 0) {
    sOut[0][0] = sOut[1][0] = 0.0;
    sOut[0][N] = sOut[1][N] = 1.0;
  }
  __syncthreads();
  if (tid < 128) wave_prefix_max(sOut[tid >> 6], N + 1, tid & 63);
  __syncthreads();
  for (int k = tid; k <= N; k += 256) {
    Gp[c * row + k] = sOut[0][k];
    Gu[c * row + k] = sOut[1][k];
  }
}

// DoSample of every child: one workgroup per (tile of A.tile points, child).
// Bound by VALU issue, with the LDS (a cell read and an FP64 add per
// coordinate) close behind.  All of a point's cells are read before the first
// is used; POW2 and FULL (d = 4 NB) as in the Vegas DoSample kernel: a
// power-of-two bin count's fraction is formed from the word's bits, and only
// the last Philox block's coordinates can be missing.
// 128 children of 2^17 points, d = 8, 128 bins, Gaussian: 116 us (145 G points/s),
// 136 with the constants in vector registers, a branch per coordinate and tiles
// of 4096 points.
template <int FAM, int NB, bool POW2, bool FULL>
__global__ void __launch_bounds__(kSuaveBlock) suave_sample_kernel(SuaveArgs A) {
  extern __shared__ __align__(16) double lds[];
  __shared__ double red[kSuaveBlock / 64];
  const int c = blockIdx.y, tile = blockIdx.x, tid = threadIdx.x;
  const int pos = A.chpos[c], serial = A.chser[c];
  const int d = A.d, N = A.N, dN = d * N;
  Cell<double> *sC = (Cell<double> *)lds;
  double *sH = lds + 2 * dN;
  const double *G = A.R.grid + (size_t)pos * d * (N + 1);
  stage_cells<double, POW2>(G, d, N, sC);
  for (int e = tid; e < dN; e += kSuaveBlock) sH[e] = 0.0;
  // the child's box and the integrand's constants, the same for the whole
  // workgroup: in scalar registers (in vector registers they take 64 at d = 8
  // and cost the fourth wavefront of a SIMD)
  constexpr int D = 4 * NB;
  double blo[D], bw[D], p0[D], p1[D], V = 1.0;
#pragma unroll
  for (int j = 0; j < D; ++j) {
    const size_t at = (size_t)pos * d + (j < d ? j : 0);
    blo[j] = uniform(A.R.lo[at]);
    bw[j] = uniform(A.R.hi[at] - A.R.lo[at]);
    p0[j] = uniform(A.p64[j]);
    p1[j] = uniform(A.p64[kParamRow + j]);
    if (j < d) V *= bw[j];
  }
  __syncthreads();
  const double phase0 = p1[0];
  const double Nd = (double)N;
  const int L = POW2 ? 31 - __clz(N) : 0;
  const double scale = pow2_scale<double>(L);
  const long long n = A.nnew;
  const long long i0 = (long long)tile * A.tile;
  const long long i1 = min(i0 + (long long)A.tile, n);
  double *vout = A.R.v + (size_t)pos * n;
  uint16_t *sout = A.R.side + (size_t)pos * n;
  double S1 = 0.0, S2 = 0.0;
  for (long long i = i0 + tid; i < i1; i += kSuaveBlock) {
    int idx[D];
    double fr[D], lo[D], sp[D];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const U4 W = philox4x32_10(
          U4{(uint32_t)i, ((uint32_t)serial << 8) | (uint32_t)b, A.sid, 0u}, A.key0, A.key1);
      const uint32_t wd[4] = {W.x, W.y, W.z, W.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = 4 * b + q;
        if (FULL || b < NB - 1 || j < d) {
          int k;
          if (POW2)
            bin_frac_pow2(wd[q], L, scale, fr[j], k);
          else
            bin_frac_any(wd[q], N, Nd, fr[j], k);
          idx[j] = j * N + k;
          const Cell<double> cell = sC[j * N + k];
          lo[j] = cell.lo;
          sp[j] = cell.span;
        }
      }
    }
    double w = 1.0;
    double acc = Genz<double, FAM>::init(phase0);
    uint32_t bits = 0;
#pragma unroll
    for (int j = 0; j < D; ++j)
      if (FULL || j < 4 * (NB - 1) || j < d) {
        const double xr = fma(fr[j], sp[j], lo[j]);
        w = POW2 ? w * sp[j] : w * (Nd * sp[j]);
        acc = Genz<double, FAM>::step(acc, fma(xr, bw[j], blo[j]), p0[j], p1[j]);
        if (xr >= 0.5) bits |= 1u << j;
      }
    const double v = (w * V) * Genz<double, FAM>::finish(acc, d);
    vout[i] = v;
    sout[i] = (uint16_t)bits;
    const double v2 = v * v;
    S1 += v;
    S2 += v2;
#pragma unroll
    for (int j = 0; j < D; ++j)
      if (FULL || j < 4 * (NB - 1) || j < d) unsafeAtomicAdd(&sH[idx[j]], v2);
  }
  S1 = block_sum(S1, red);
  S2 = block_sum(S2, red);
  const size_t t = (size_t)c * A.ntiles + tile;
  if (tid == 0) {
    A.tsum[2 * t] = S1;
    A.tsum[2 * t + 1] = S2;
  }
  __syncthreads();
  for (int e = tid; e < dN; e += kSuaveBlock) A.thist[t * dN + e] = sH[e];
}

// One workgroup per (child, dimension): the refined grid of the dimension;
// dimension 0's also takes the child's own estimate and the combination.
// Latency: the tile rows of N bins in one trip, then the refinement's chain.
// 128 children, d = 8, 128 bins: 10.9 us, 14.7 with one workgroup per child.
constexpr int kSuaveFold = 256;  // threads (and at most kMaxBins = 256 bins)

__global__ void __launch_bounds__(kSuaveFold) suave_fold_kernel(SuaveArgs A) {
  __shared__ double H[kMaxBins], D[kMaxBins], E[kMaxBins + 1];
  __shared__ double red[kSuaveFold / 64];
  const int c = blockIdx.x, j = blockIdx.y, tid = threadIdx.x;
  const int pos = A.chpos[c];
  const int d = A.d, N = A.N, dN = d * N, row = N + 1, nt = A.ntiles;
  const bool refine = !(A.flags & FLAG_FREEZE_GRID);
  double *G = A.R.grid + ((size_t)pos * d + j) * row;
  if (refine) {
    const double *th = A.thist + (size_t)c * nt * dN + (size_t)j * N + tid;
    if (tid < N) {
      double h = 0.0;
#pragma unroll 16
      for (int t = 0; t < nt; ++t) h += th[(size_t)t * dN];
      H[tid] = h;
    }
    for (int e = tid; e < row; e += kSuaveFold) E[e] = G[e];
  }
  if (j == 0) {
    double S1 = 0.0, S2 = 0.0;
    for (int t = tid; t < nt; t += kSuaveFold) {
      S1 += A.tsum[2 * ((size_t)c * nt + t)];
      S2 += A.tsum[2 * ((size_t)c * nt + t) + 1];
    }
    S1 = block_sum(S1, red);
    S2 = block_sum(S2, red);
    if (tid == kSuaveFold - 1) {  // (not the wavefront that refines)
      const double n = (double)A.nnew;
      const double I = S1 / n;
      const double var = fmax(0.0, S2 / n - I * I) / (n - 1.0);
      const double iI = A.R.inh_I[pos], iv = A.R.inh_var[pos];
      const bool inh = iv > 0.0;
      const double Ik[2] = {iI, I}, Vk[2] = {iv, var};
      const int k0 = inh ? 0 : 1;
      int nzero = 0;
      double zsum = 0.0;
      for (int k = k0; k < 2; ++k)
        if (Vk[k] == 0.0) {
          ++nzero;
          zsum += Ik[k];
        }
      double Ir, Vr, chi2 = 0.0;
      if (nzero > 0) {
        Ir = zsum / nzero;
        Vr = 0.0;
      } else {
        double ws = 0.0, wi = 0.0;
        for (int k = k0; k < 2; ++k) {
          ws += 1.0 / Vk[k];
          wi += Ik[k] / Vk[k];
        }
        Ir = wi / ws;
        Vr = 1.0 / ws;
        for (int k = k0; k < 2; ++k) chi2 += (Ik[k] - Ir) * (Ik[k] - Ir) / Vk[k];
      }
      A.R.I[pos] = Ir;
      A.R.var[pos] = Vr;
      A.R.chi2[pos] = chi2;
      A.R.dof[pos] = inh ? 1 : 0;
    }
  }
  __syncthreads();
  if (refine && tid < 64) rebin_dimension(H, D, E, G, N, tid);
}

// Totals over the R regions (fixed order), the stop rule's outcome and, once
// the run ends with them, the chi^2 probability.  The outcome goes to the
// host as one word, seq << 8 | code, that it polls (code 0: go on, 1:
// accuracy reached, 2: not finite); the totals beside it are read after the
// stream has drained.
__global__ void __launch_bounds__(1024) suave_totals_kernel(SuaveArgs A, int R, SStop stop) {
  __shared__ double red[4][16];
  const int tid = threadIdx.x;
  const int chunk = (R + 1023) / 1024;
  const int b0 = min(tid * chunk, R), b1 = min(b0 + chunk, R);
  double x[4] = {0.0, 0.0, 0.0, 0.0};
  for (int i = b0; i < b1; ++i) {
    x[0] += A.R.I[i];
    x[1] += A.R.var[i];
    x[2] += A.R.chi2[i];
    x[3] += (double)A.R.dof[i];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    x[k] = wave_sum(x[k]);
    if ((tid & 63) == 0) red[k][tid >> 6] = x[k];
  }
  __syncthreads();
  if (tid == 0) {
    double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      for (int q = 0; q < 16; ++q) t[k] += red[k][q];
    SState st;
    st.I = t[0];
    st.var = t[1];
    st.chi2 = t[2];
    st.dof = (int)t[3];
    st.pad = 0;
    int code = 0;
    if (!isfinite(st.I) || !isfinite(st.var))
      code = 2;
    else if (stop.neval >= stop.mineval &&
             sqrt(st.var) <= fmax(stop.epsabs, stop.epsrel * fabs(st.I)))
      code = 1;
    st.prob = (code || stop.last) && st.dof > 0 ? gamma_p(0.5 * st.dof, 0.5 * st.chi2) : 0.0;
    *stop.state = st;
    __hip_atomic_store(stop.word, ((unsigned long long)stop.seq << 8) | (unsigned long long)code,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// ---- launchers ---------------------------------------------------------------

size_t suave_sample_lds(int d, int N) { return (size_t)3 * d * N * sizeof(double); }

hipError_t launch_suave_root(const SuaveArgs &A, hipStream_t s) {
  hipLaunchKernelGGL(suave_root_kernel, dim3(1), dim3(256), 0, s, A);
  return hipGetLastError();
}

hipError_t launch_topk(const double *key, int R, int K, int *sel, hipStream_t s) {
  hipLaunchKernelGGL(topk_kernel, dim3(1), dim3(1024), 0, s, key, R, K, sel);
  return hipGetLastError();
}

hipError_t launch_suave_select(const SuaveArgs &A, int R, int K, hipStream_t s) {
  return launch_topk(A.R.var, R, K, A.sel, s);
}

hipError_t launch_suave_fluct(const SuaveArgs &A, int K, hipStream_t s) {
  const dim3 grid(A.nchunks, K), block(kFlThreads * ((A.d + kFlDims - 1) / kFlDims));
  hipLaunchKernelGGL(suave_fluct1_kernel, grid, block, 0, s, A);
  hipLaunchKernelGGL(suave_fluct2_kernel, grid, block, 0, s, A);
  return hipGetLastError();
}

hipError_t launch_suave_split(const SuaveArgs &A, int R, long long Q, int K, hipStream_t s) {
  hipLaunchKernelGGL(suave_split_kernel, dim3(K), dim3(256), 0, s, A, R, Q);
  return hipGetLastError();
}

namespace {

template <int FAM, int NB>
void launch_sample_nb(const SuaveArgs &A, dim3 grid, size_t lds, hipStream_t s) {
  const bool pow2 = (A.N & (A.N - 1)) == 0, full = A.d == 4 * NB;
  const auto kernel = pow2 ? (full ? suave_sample_kernel<FAM, NB, true, true>
                                   : suave_sample_kernel<FAM, NB, true, false>)
                           : (full ? suave_sample_kernel<FAM, NB, false, true>
                                   : suave_sample_kernel<FAM, NB, false, false>);
  // more LDS than a launch gets by default (up to d = 16 with 256 bins); a
  // runtime that refuses keeps its limit, and the launch reports an error
  if (lds > 64 * 1024 &&
      hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                          160 * 1024) != hipSuccess)
    (void)hipGetLastError();
  hipLaunchKernelGGL(kernel, grid, dim3(kSuaveBlock), lds, s, A);
}

template <int FAM>
void launch_sample_fam(const SuaveArgs &A, dim3 grid, size_t lds, hipStream_t s) {
  switch ((A.d + 3) / 4) {
    case 1: launch_sample_nb<FAM, 1>(A, grid, lds, s); break;
    case 2: launch_sample_nb<FAM, 2>(A, grid, lds, s); break;
    case 3: launch_sample_nb<FAM, 3>(A, grid, lds, s); break;
    default: launch_sample_nb<FAM, 4>(A, grid, lds, s); break;
  }
}

}  // namespace

hipError_t launch_suave_sample(const SuaveArgs &A, int nchild, hipStream_t s) {
  const dim3 grid(A.ntiles, nchild);
  const size_t lds = suave_sample_lds(A.d, A.N);
  switch (A.family) {
    case GAUSSIAN:
      launch_sample_fam<GAUSSIAN>(A, grid, lds, s);
      break;
    case OSCILLATORY:
      launch_sample_fam<OSCILLATORY>(A, grid, lds, s);
      break;
    case PRODUCT_PEAK:
      launch_sample_fam<PRODUCT_PEAK>(A, grid, lds, s);
      break;
    case CORNER_PEAK:
      launch_sample_fam<CORNER_PEAK>(A, grid, lds, s);
      break;
    default:
      launch_sample_fam<C0>(A, grid, lds, s);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_suave_fold(const SuaveArgs &A, int nchild, hipStream_t s) {
  const int dims = A.flags & FLAG_FREEZE_GRID ? 1 : A.d;
  hipLaunchKernelGGL(suave_fold_kernel, dim3(nchild, dims), dim3(kSuaveFold), 0, s, A);
  return hipGetLastError();
}

hipError_t launch_suave_totals(const SuaveArgs &A, int R, const SStop &stop, hipStream_t s) {
  hipLaunchKernelGGL(suave_totals_kernel, dim3(1), dim3(1024), 0, s, A, R, stop);
  return hipGetLastError();
}

}  // namespace ccuba
