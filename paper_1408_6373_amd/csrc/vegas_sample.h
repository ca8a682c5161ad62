// vegas_sample.h -- the Vegas DoSample kernel (a1-a6) and the
// per-coordinate helpers it shares with the points kernel.
//
// The kernel template is instantiated per precision and histogram type in
// its own translation unit (vegas_sample_*.hip), so that the instances build
// in parallel; vegas.hip dispatches to them.
#pragma once
#ifndef CCUBA_RTC  // the run-time compiled build has no C++ library headers
#include <cstddef>
#include <vector>
#else
#define offsetof(type, member) __builtin_offsetof(type, member)
#endif

#include "engine.h"
#include "genz.h"
#include "philox.h"
#include "vegas.h"

namespace ccuba {

// ---------------------------------------------------------------------------
// Descriptors read as one word per lane: a single vector load brings a whole
// VJob (or VState) into the wavefront, where field-by-field scalar loads are
// issued as each field is first needed and can each cost a round trip to
// memory.  Lanes past the descriptor's last word read nothing.
constexpr int kJobWords = (int)(sizeof(VJob) / 4);
constexpr int kStateWords = (int)(sizeof(VState) / 4);
static_assert(sizeof(VJob) % 8 == 0 && kJobWords <= 64, "a VJob fits one wavefront");
static_assert(sizeof(VState) % 8 == 0 && kStateWords <= 64, "a VState fits one wavefront");

template <int NW>
__device__ __forceinline__ uint32_t load_words(const void *p, int lane) {
  return lane < NW ? ((const __attribute__((address_space(1))) uint32_t *)p)[lane] : 0u;
}

// The field at byte offset OFF of the descriptor whose words the wavefront
// holds (a wave-uniform value).
template <typename F, int OFF>
__device__ __forceinline__ F word_field(uint32_t w) {
  static_assert(OFF % 4 == 0 && (sizeof(F) == 4 || sizeof(F) == 8), "word-aligned field");
  if constexpr (sizeof(F) == 4) {
    const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)w, OFF / 4);
    F r;
    __builtin_memcpy(&r, &v, 4);
    return r;
  } else {
    const unsigned long long v =
        (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)w, OFF / 4) |
        ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)w, OFF / 4 + 1) << 32);
    F r;
    __builtin_memcpy(&r, &v, 8);
    return r;
  }
}
#define JOB_FIELD(w, f) (word_field<decltype(VJob::f), (int)offsetof(VJob, f)>(w))

// The whole descriptor from the words the wavefront holds (the reads of
// fields the caller never uses are dropped).
template <typename S>
__device__ __forceinline__ S from_words(uint32_t w) {
  constexpr int n = (int)(sizeof(S) / 4);
  uint32_t words[n];
#pragma unroll
  for (int i = 0; i < n; ++i) words[i] = (uint32_t)__builtin_amdgcn_readlane((int)w, i);
  S r;
  __builtin_memcpy(&r, words, sizeof(S));
  return r;
}

// A device pointer taken from a descriptor word is a generic pointer, and
// loads through it are flat loads, which also count against the scalar
// memory counter: a wait for any scalar load then waits for them too.
// Loads through the global-address-space view are global loads.
template <typename T>
using gbl = __attribute__((address_space(1))) T;
template <typename T>
__device__ __forceinline__ const gbl<T> *gload(const T *p) {
  return (const gbl<T> *)p;
}
template <typename T>
__device__ __forceinline__ gbl<T> *gstore(T *p) {
  return (gbl<T> *)p;
}

// The value lane l of the wavefront holds (l wave-uniform).
__device__ __forceinline__ double lane_value(double v, int l) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// a3: the grid as staged in LDS.  Cell k of dimension j sits at [j * N + k]
// and holds its lower edge and its span in the working precision: the width
// E[k+1] - E[k] for a general N, and N times the width when N = 2^L.  Both
// are formed once per tile from the two converted edges, exactly as they
// would be formed per point (scaling by 2^L is exact), so staging changes no
// value.  One LDS read per coordinate fetches both.

template <typename T>
struct alignas(2 * sizeof(T)) Cell {
  T lo, span;
};

// Each thread loads the edges of kStageCells cells before it stores any, so
// that the whole grid of a typical integral (up to kStageCells * blockDim
// cells) arrives in one round trip to memory.  Indices past the end are
// clamped to the last cell: their loads stay in range and nothing is stored.
constexpr int kStageCells = 4;

template <typename T, bool POW2>
__device__ __forceinline__ void stage_cells(const double *__restrict__ E, int d, int N,
                                            Cell<T> *sC) {
  const int row = N + 1, dN = d * N, bs = blockDim.x;
  const T Nt = (T)N;
  const gbl<double> *Eg = gload(E);
  auto batch = [&](int e0) {
    double lo[kStageCells], hi[kStageCells];
#pragma unroll
    for (int b = 0; b < kStageCells; ++b) {
      const int e = min(e0 + b * bs, dN - 1), j = e / N, k = e - j * N;
      lo[b] = Eg[j * row + k];
      hi[b] = Eg[j * row + k + 1];
    }
#pragma unroll
    for (int b = 0; b < kStageCells; ++b) {
      const int e = e0 + b * bs;
      const T l = (T)lo[b], h = (T)hi[b];
      if (e < dN) sC[e] = Cell<T>{l, POW2 ? Nt * (h - l) : h - l};
    }
  };
  // the first batch outside the loop: a loop head would wait for every load
  // in flight (the caller's too) before reusing the batch's registers
  batch(threadIdx.x);
  for (int e0 = threadIdx.x + kStageCells * bs; e0 < dN; e0 += kStageCells * bs) batch(e0);
}

// The sum over the wavefront, in every lane: the butterfly over lane distances
// 32, 16, ..., 1 (so the same pairs are added as with exchanges by lane
// index), without LDS traffic: row swaps bring the halves and the rows
// together, then each row holds all sums and rotates.
template <int CTRL>
__device__ __forceinline__ double row_rotated(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double wave_sum(double v) {
  {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32),
                                                    false, false);
    v = __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
        __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
  }
  {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32),
                                                    false, false);
    v = __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
        __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
  }
  v += row_rotated<0x128>(v);  // row_ror:8
  v += row_rotated<0x124>(v);  // (lanes equal mod 8 hold the same value)
  v += row_rotated<0x122>(v);
  v += row_rotated<0x121>(v);
  return v;
}


// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ float uniform(float v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(v)));
}
__device__ __forceinline__ double uniform(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readfirstlane((int)b);
  const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

template <typename T>
__device__ __forceinline__ const T *param_ptr(const VJob &J, int which);
template <>
__device__ __forceinline__ const double *param_ptr<double>(const VJob &J, int which) {
  return J.p64 + which * kParamRow;
}
template <>
__device__ __forceinline__ const float *param_ptr<float>(const VJob &J, int which) {
  return J.p32 + which * kParamRow;
}

__device__ __forceinline__ double fma_t(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return fmaf(a, b, c); }

// Bin and fractional position of one coordinate (a2 + the first half of
// a3).  General N: z = y N, k = min(floor z, N - 1), frac = z - k, then
// x = fma(frac, width, lo) and w *= N width.
// N = 2^L: the bin is the top L bits of the word and the fraction the bits
// below them, which is exactly what the floating-point formula gives (every
// step there is exact).  These helpers return fs = frac / N (exact), so that
// with the staged span s = N width, x = fma(fs, s, lo) has the same exact
// product fs s = frac width and rounds to the same x, and w *= s is the same
// product as before: one multiply fewer per coordinate.
__device__ __forceinline__ void bin_frac_pow2(uint32_t r, int L, double scale, double &fs,
                                              int &k) {
  k = (int)(r >> (32 - L));
  const uint32_t m = (r << L) | (1u << (L - 1));  // (r N mod 2^32) + N/2
  fs = (double)m * scale;                         // scale = 2^(-32-L)
}
__device__ __forceinline__ void bin_frac_pow2(uint32_t r, int L, float scale, float &fs,
                                              int &k) {
  k = (int)(r >> (32 - L));
  // the 23 - L bits of r >> 9 below the bin index, then the half-step bit
  // 2^(L-1), as the mantissa M of a float with exponent -L: that float is
  // 2^-L (1 + M 2^-23), and removing 2^-L (= scale) leaves M 2^(-23-L)
  // = frac / N exactly.  (x & mask) | c is one three-input bit operation
  // (truth table 0xEA).
  static_assert(kMaxBins <= 512, "the shift below needs L <= 9");
  const uint32_t mask = 0x7FFFFFu & ~((1u << L) - 1u);
  const uint32_t c = ((uint32_t)(127 - L) << 23) | (1u << (L - 1));
  const uint32_t bits = (uint32_t)__builtin_amdgcn_bitop3_b32(r >> (9 - L), mask, c, 0xEA);
  fs = __uint_as_float(bits) - scale;
}
__device__ __forceinline__ void bin_frac_any(uint32_t r, int N, double Nd, double &frac, int &k) {
  const double y = (double)r * 0x1p-32 + 0x1p-33;
  const double z = y * Nd;
  int kk = (int)z;
  kk = kk > N - 1 ? N - 1 : kk;
  frac = z - (double)kk;
  k = kk;
}
__device__ __forceinline__ void bin_frac_any(uint32_t r, int N, float Nf, float &frac, int &k) {
  const float y = (float)(r >> 9) * 0x1p-23f + 0x1p-24f;
  const float z = y * Nf;
  int kk = (int)z;
  kk = kk > N - 1 ? N - 1 : kk;
  frac = z - (float)kk;
  k = kk;
}

// 2^-L (FP32) or 2^(-32-L) (FP64): the scale of the power-of-two fraction.
template <typename T>
__device__ __forceinline__ T pow2_scale(int L);
template <>
__device__ __forceinline__ float pow2_scale<float>(int L) {
  return __uint_as_float((uint32_t)(127 - L) << 23);
}
template <>
__device__ __forceinline__ double pow2_scale<double>(int L) {
  return __longlong_as_double((long long)(1023 - 32 - L) << 52);
}

// ---------------------------------------------------------------------------
// a6: the histogram in 64-bit fixed point, exactly.
//
// LDS integer adds are several times cheaper than FP64 adds on gfx950 (and
// FP32 LDS atomics far slower still).  With FP32 evaluation every v^2 has a
// 24-bit mantissa, so a v^2 that is a whole multiple of a unit 2^(E-62) goes
// into an unsigned 64-bit sum without any rounding; 2^E bounds the tile's
// total of every bin, so the sums cannot overflow, and integer sums do not
// depend on the order of the adds.  Every other v^2 -- too small to be a
// whole multiple of the unit, above the cap, or not finite -- goes to a
// second, FP64 histogram, as on the FP64 path.  The two are added when the
// tile is written, so the tile's histogram is the FP64 one up to rounding
// order: the split changes speed, not results.
//
// The bound is 2^E >= 4 cnt c for the tile's cnt points and a cap c on the
// v^2 that may enter the fixed-point sums.  In an integral's first
// iteration c is a true bound from the staged grid and the integrand's
// maximum: w <= prod_j max_k (N width_jk), and f <= 1 for every family except
// the product peak, where f <= 1 / prod_j a_j^-2 (the FP32 products are
// formed in the order the point's own products are, so rounding keeps them
// bounds).  Once the grid adapts that bound grows far beyond the values that
// occur (it takes every dimension's widest bin), so later iterations take
// c = 1024 times the mean v^2 of the previous one (at most 1 in 1024 of the
// v^2 exceed that).
//
// With FP64 evaluation v^2 has a 53-bit mantissa M, v^2 = M 2^(e - 1075) for
// the biased exponent e.  In units U = 2^(E - 91) it is the integer
// X = M 2^s, s = e - 984 - E, whenever s >= 0, and X < 2^90: its low 32 bits
// and X >> 32 go to two 64-bit sums (below 2^46 and 2^57 for a tile of any
// size), so the FP64 histogram too is exact and does not depend on the order
// of the adds, for two integer LDS adds that cost about what one FP64 LDS
// add does.  Every other v^2 goes to the FP64 histogram beside them.

template <typename HT>
struct FixedHist {
  static constexpr bool value = false;
};
template <>
struct FixedHist<unsigned long long> {
  static constexpr bool value = true;
};

// The LDS layout of an instance.  For a power-of-two bin count the histogram
// comes first, in a region of ND * kMaxBins bins whatever d and N are, and the
// cells start at its end: both then lie at offsets that are known when the
// kernel is compiled, so that one address per coordinate (two instructions from
// the word) serves the FP32 cell and the histogram bin alike, the rest being the
// instructions' own offsets.  The FP64 histogram beside a
// fixed-point one (rarely touched) takes the part of the region that N <= 128
// leaves, or follows the cells.  Other bin counts, and the two-word fixed-point
// histogram, take the cells first and everything without gaps.
// Two integrals of 20 x 10^7 points at d = 8, 128 bins, FP32: 2.41 ms, 2.43 ms with
// the compact layout and separate addresses (120 vector registers against 134;
// 196 vector instructions per point, 90% of their issue rate).
template <typename T, typename HT, int NB, bool POW2>
struct LdsLayout {
  static constexpr bool kFixed = FixedHist<HT>::value;
  static constexpr bool kConst = POW2 && !(kFixed && sizeof(T) == 8);
  static constexpr int kRegion = 4 * NB * kMaxBins * 8;  // bytes of the histogram's region
};

template <int V>
struct Int {
  static constexpr int value = V;
};

// LDS by address: what lies at a byte address, and the address of an object.
template <typename V>
__device__ __forceinline__ V *lds_at(uint32_t a) {
  return (V *)(__attribute__((address_space(3))) V *)(unsigned long long)a;
}
template <typename V>
__device__ __forceinline__ uint32_t lds_addr(V *p) {
  return (uint32_t)(unsigned long long)(__attribute__((address_space(3))) V *)p;
}

// Sample the points [i0, i0 + cnt) of one tile; lane sums of v - shift and
// (v - shift)^2 go to S1, S2.
// NB = ceil(d/4) Philox blocks per point and the R = d - 4 (NB - 1) coordinates
// of the last one are template arguments, so that the per-dimension loops are
// unrolled without a branch on d in them (R = 0: read from the descriptor, for
// callers' functions, whose compile time the caller waits for).  10 iterations of
// 4 x 10^6 points at d = 7, 100 bins, FP64: 567 us, 592 with a test per coordinate
// of the last block.
// Each lane carries ILP independent points per trip (q, q + blockDim, ...),
// so that several Philox chains are in flight; what is left at the tile's end goes
// one point at a time (a caller's function, of any size, is compiled once: its last
// trip computes past the end).  A trip's
// histogram updates are issued at its end, so that the LDS works through
// them while the next trip's Philox rounds run; the next trip's wait for its
// grid reads then finds them done.  (Updates deferred to after the next
// trip's grid reads made every such wait also wait for the updates.)
template <typename T, typename HT, int FAM, int NB, int ILP, bool POW2, int R>
__device__ __forceinline__ void sample_tile(const VJob &J, int t, long long i0, int cnt,
                                            const Cell<T> *__restrict__ sC, HT *sH,
                                            const T (&pp0)[4 * NB], const T (&pp1)[4 * NB],
                                            int E, float cap, double shift,
                                            double *sHx, double &S1, double &S2) {
  constexpr int ND = 4 * NB;
  const int d = R ? 4 * (NB - 1) + R : J.ndim, N = J.nbins;
  const T Nt = (T)N;
  const int L = POW2 ? 31 - __clz(N) : 0;
  const T scale = pow2_scale<T>(L);
  const uint32_t c1 = (uint32_t)t << 8;
  const uint32_t sid = J.sid, k0 = J.key0, k1 = J.key1;
#ifndef CCUBA_RTC
  const T phase0 = pp1[0];
#endif
  constexpr bool CL = LdsLayout<T, HT, NB, POW2>::kConst;
  const uint32_t lds0 = CL ? lds_addr(sH) : 0;
  const int bs = blockDim.x;
  // an assembly comment naming the family, so that the per-point loop that
  // follows can be found in the assembly listing (it emits no instruction)
  asm volatile("; ccuba sample_tile family %0" ::"n"(FAM));
  // one trip: P points per lane from q0 on (with MASK, those past the tile's end
  // are computed too, with LDS reads in range, and contribute nothing)
  auto trip = [&](int q0, auto points, auto mask) {
    constexpr int P = decltype(points)::value;
    constexpr bool MASK = decltype(mask)::value;
    T fr[P][ND], lo[P][ND], sp[P][ND];
    int idx[P][ND];
    // words, bins and the grid cells they select
#pragma unroll
    for (int e = 0; e < P; ++e) {
      const uint32_t i = (uint32_t)(i0 + q0 + e * bs);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const U4 r = philox4x32_10(U4{i, c1 | (uint32_t)b, sid, 0u}, k0, k1);
        const uint32_t rr[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int j = 4 * b + c;
          if (b < NB - 1 || j < d) {
            int k;
            if (POW2)
              bin_frac_pow2(rr[c], L, scale, fr[e][j], k);
            else
              bin_frac_any(rr[c], N, Nt, fr[e][j], k);
            // constant layout: FP32 keeps the address, which serves both; FP64,
            // whose cells are twice as wide, the bin
            idx[e][j] = !CL              ? j * N + k
                        : sizeof(T) == 4 ? (int)(((uint32_t)k << 3) + (lds0 + 8u * j * N))
                                         : k;
            const Cell<T> cell =
                !CL              ? sC[idx[e][j]]
                : sizeof(T) == 4 ? *lds_at<Cell<T>>(
                                       (uint32_t)idx[e][j] + LdsLayout<T, HT, NB, POW2>::kRegion)
                                 : *lds_at<Cell<T>>(
                                       ((uint32_t)k << 4) +
                                       (lds0 + LdsLayout<T, HT, NB, POW2>::kRegion + 16u * j * N));
            lo[e][j] = cell.lo;
            sp[e][j] = cell.span;
          }
        }
      }
    }
    // weights, integrand, sums, histogram updates
#pragma unroll
    for (int e = 0; e < P; ++e) {
      T w = (T)1;
#ifdef CCUBA_RTC
      // a caller's function of the whole point, compiled with this kernel:
      // T ccuba_user(const T *x, int ndim, const T *a, const T *u)
      T xs[ND];
#pragma unroll
      for (int j = 0; j < ND; ++j) {
        if (j < 4 * (NB - 1) || j < d) {
          xs[j] = fma_t(fr[e][j], sp[e][j], lo[e][j]);
          w = POW2 ? w * sp[e][j] : w * (Nt * sp[e][j]);
        } else {
          xs[j] = (T)0;
        }
      }
      const T v = w * ccuba_user(xs, d, pp0, pp1);
#else
      T acc = Genz<T, FAM>::init(phase0);
#pragma unroll
      for (int j = 0; j < ND; ++j) {
        if (j < 4 * (NB - 1) || j < d) {
          const T x = fma_t(fr[e][j], sp[e][j], lo[e][j]);
          w = POW2 ? w * sp[e][j] : w * (Nt * sp[e][j]);
          acc = Genz<T, FAM>::step(acc, x, pp0[j], pp1[j]);
        }
      }
      const T v = w * Genz<T, FAM>::finish(acc, d);
#endif
      // the bin of coordinate j in the histogram, and in the FP64 one beside it
      auto bin = [&](int j) {
        if constexpr (!CL)
          return sH + idx[e][j];
        else if constexpr (sizeof(T) == 4)
          return lds_at<HT>((uint32_t)idx[e][j]);
        else
          return lds_at<HT>(((uint32_t)idx[e][j] << 3) + (lds0 + 8u * j * N));
      };
      auto bin_x = [&](int j) {
        return CL ? lds_at<double>((uint32_t)idx[e][j] + (lds_addr(sHx) - lds0))
                  : sHx + idx[e][j];
      };
      if (MASK && q0 + e * bs >= cnt) continue;
      const double dv = (double)v - shift;
      S1 += dv;
      S2 = fma(dv, dv, S2);
      if constexpr (FixedHist<HT>::value && sizeof(T) == 8) {
        const double v2 = v * v;
        const unsigned long long b = (unsigned long long)__double_as_longlong(v2);
        const int eb = (int)(b >> 52);
        const int s = eb - (984 + E);  // v2 = M 2^s units; s <= 37 below the cap
        if (v2 <= (double)cap && s >= 0 && eb >= 1) {
          const unsigned long long M = (b & 0xFFFFFFFFFFFFFull) | (1ull << 52);
          const unsigned long long xlo = (M << s) & 0xFFFFFFFFull;
          const unsigned long long xhi = (M << 11) >> (43 - s);  // floor(M 2^(s-32))
          HT *sHh = sH + d * N;
#pragma unroll
          for (int j = 0; j < ND; ++j)
            if (j < 4 * (NB - 1) || j < d) {
              atomicAdd(bin(j), xlo);
              atomicAdd(sHh + idx[e][j], xhi);
            }
        } else {  // not a normal whole multiple of the unit, above the cap, or not finite
#pragma unroll
          for (int j = 0; j < ND; ++j)
            if (j < 4 * (NB - 1) || j < d) unsafeAtomicAdd(bin_x(j), v2);
        }
      } else if constexpr (FixedHist<HT>::value) {
        const float v2f = (float)(v * v);
        const uint32_t b = __float_as_uint(v2f);
        const int sh = (int)(b >> 23) - (88 + E);  // v2 = m 2^sh units
        if (v2f <= cap && sh >= 0 && b >= 0x800000u) {  // (zeros and subnormals: below)
          const unsigned long long v2 = (unsigned long long)((b & 0x7FFFFFu) | 0x800000u)
                                        << sh;
#pragma unroll
          for (int j = 0; j < ND; ++j)
            if (j < 4 * (NB - 1) || j < d) atomicAdd(bin(j), v2);
        } else {  // not a normal whole multiple of the unit, above the cap, or not finite
          const double v2 = (double)v2f;
#pragma unroll
          for (int j = 0; j < ND; ++j)
            if (j < 4 * (NB - 1) || j < d) unsafeAtomicAdd(bin_x(j), v2);
        }
      } else {
        const HT v2 = (HT)(v * v);
#pragma unroll
        for (int j = 0; j < ND; ++j)
          if (j < 4 * (NB - 1) || j < d) unsafeAtomicAdd(bin(j), v2);
      }
    }
  };
  int q0 = threadIdx.x;
#ifdef CCUBA_RTC
  for (; q0 < cnt; q0 += ILP * bs) trip(q0, Int<ILP>{}, Int<(ILP > 1)>{});
#else
  if constexpr (ILP > 1)
    for (int end = ILP * bs; end <= cnt; end += ILP * bs, q0 += ILP * bs)
      trip(q0, Int<ILP>{}, Int<0>{});
  for (; q0 < cnt; q0 += bs) trip(q0, Int<1>{}, Int<0>{});
#endif
}

// One kernel per (precision, histogram type, ILP, NB, power-of-two bins,
// d = 4 NB): every instance only holds the registers and the tests its own
// class needs.  A launch walks the slice [tile_first, tile_first +
// tile_count) of the tile list, which holds the tiles of the jobs of that
// class.
// FP32 with power-of-two bins is held to the registers of four waves per SIMD
// (three above 12 dimensions), so that blocks of a batch's two halves run beside
// each other: 256 integrals of 10^4 to 10^6 points, d = 2 to 12, in 4.06 ms instead
// of 4.22 with 139 registers at d = 9 to 12.  (A few values used outside the loops
// are spilled.)  A caller's function takes the registers that it needs: what it
// holds of a point is not known here.  Three arrays of 16 words, 10 x 8 x 10^6
// points: 3.1 ms at d = 12, 7.0 with 68 registers spilled under the bound.
#ifdef CCUBA_RTC
constexpr int sample_waves(bool, int) { return 1; }
#else
constexpr int sample_waves(bool f32_pow2, int nb) { return !f32_pow2 ? 1 : nb == 4 ? 3 : 4; }
#endif

template <typename T, typename HT, int ILP, int NB, bool POW2, bool FULL>
__global__ void __launch_bounds__(256, sample_waves(sizeof(T) == 4 && POW2, NB))
    vegas_dosample_kernel(VegasArgs A) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double red[2][4];
  __shared__ uint32_t smax[kMaxDim + 2];  // fixed-point histogram: per-dimension maxima, E, cap
  using Layout = LdsLayout<T, HT, NB, POW2>;
  Cell<T> *sC = (Cell<T> *)(smem + (Layout::kConst ? Layout::kRegion : 0));
  HT *sH = (HT *)(smem + (Layout::kConst ? 0 : A.lds_hist_byte_off));
  const int tid = threadIdx.x, bs = blockDim.x, lane = tid & 63, wid = tid >> 6;
  const int myprec = sizeof(T) == 8 ? FP64 : FP32;

  const int tend = A.tile_first + A.tile_count;
  for (int tt = A.tile_first + blockIdx.x; tt < tend; tt += gridDim.x) {
    // the descriptor as one vector load (a word per lane); with one job in
    // the launch its index needs no lookup
    const int jb = A.njobs == 1 ? 0 : A.tile_job[tt];
    const VJob J = from_words<VJob>(load_words<kJobWords>(A.jobs + jb, lane));
    if (J.prec != myprec || ((J.ndim + 3) >> 2) != NB ||
        ((J.nbins & (J.nbins - 1)) == 0) != POW2 || (FULL && J.ndim != 4 * NB))
      continue;
    const int d = J.ndim, N = J.nbins, dN = d * N;
    // One round trip to memory for: the state (a word per lane), the
    // integrand's parameters (rows zero-padded to 16) and the grid cells
    // (staged into LDS whether or not the integral turns out to be done).
    uint32_t sw = load_words<kStateWords>(J.state, lane);
    constexpr int ND = 4 * NB;
    T pp0[ND], pp1[ND];
    {
      const gbl<T> *p0 = gload(param_ptr<T>(J, 0)), *p1 = gload(param_ptr<T>(J, 1));
#pragma unroll
      for (int j = 0; j < ND; ++j) {
        pp0[j] = p0[j];
        pp1[j] = p1[j];
      }
    }
    stage_cells<T, POW2>(J.grid, d, N, sC);
    // the state words are first used here, after the cells' loads are issued
    // (without this the compiler waits for them before issuing those loads)
    asm volatile("" : "+v"(sw)::"memory");
    const int lt = tt - J.tile0;
    // the state as this iteration samples it, for the refine launch (also once
    // the integral is done)
    if (J.snap && lt == 0 && wid == 0 && lane < kStateWords) ((uint32_t *)J.snap)[lane] = sw;
    const VState st = from_words<VState>(sw);
    if (st.done) continue;  // the same for the whole block: nothing read the cells yet
    // (only now: their loads have been in flight beside the cells').  FP32 at up
    // to 8 dimensions keeps them in vector registers: it has those to spare,
    // and an instruction reads one scalar operand.  So do FP64 above 12 dimensions,
    // where the scalar registers hold a part of them only, and above 8 with
    // power-of-two bins (other bin counts would pass the 256 registers of two
    // wavefronts a SIMD), but for the fixed-point histogram: 3 iterations of
    // 3 x 10^7 points of the continuous family at d = 16, 256 bins, 1818 us with
    // scalar ones, 1659 now; at d = 12, 6 x 10^6 points, 398 and 336; a Gaussian at
    // d = 12, 100 bins, 3 x 10^7 points, 1222 and 1319 (so scalar there).  And so does a
    // caller's function, whose loops may index them: 10 x 2 x 10^7 points of a Gaussian's
    // loop at d = 11, FP32, 2.3 ms, 2.9 with scalar ones.
#ifndef CCUBA_RTC
    constexpr bool kVector = sizeof(T) == 4 ? NB <= 2
                                            : !Layout::kFixed && (NB == 4 || (NB == 3 && POW2));
    if constexpr (!kVector) {
#pragma unroll
      for (int j = 0; j < ND; ++j) {
        pp0[j] = uniform(pp0[j]);
        pp1[j] = uniform(pp1[j]);
      }
    }
#endif
    const long long n_t = J.nstart + (long long)st.T * J.nincrease;
    // The tiles are sized for the run's largest iteration; a smaller one is
    // spread over all of them (whole trips of the block), so that its launch
    // is as short as its points allow: every tile's row is written anyhow.
    // A run to 1e-4 at d = 6 from 10^5 points an iteration, tiles planned for
    // 6.9e5: 166 us, 177 with the first iterations in the first tiles.
    uint32_t per = (uint32_t)n_t / (uint32_t)J.ntiles;  // (n_t < 2^32)
    if ((long long)per * J.ntiles < n_t) ++per;
    long long span = ((long long)per + bs - 1) / bs * bs;
    span = span < J.tile_pts ? span : J.tile_pts;
    const long long i0 = (long long)lt * span;
    long long c = n_t - i0;
    c = c < 0 ? 0 : (c > span ? span : c);
    const int cnt = (int)c;

    // fixed point: the integer sums (two per bin with FP64 evaluation), then
    // the FP64 histogram of the rest
    constexpr int kFixWords = (FixedHist<HT>::value && sizeof(T) == 8) ? 2 : 1;
    for (int e = tid; e < kFixWords * dN; e += bs) sH[e] = (HT)0;
    double *sHx = (double *)(sH + kFixWords * dN);
    if constexpr (Layout::kConst)
      if (2 * dN * 8 > Layout::kRegion) sHx = (double *)(sC + dN);
    if constexpr (FixedHist<HT>::value) {
      for (int e = tid; e < dN; e += bs) sHx[e] = 0.0;
      if (tid <= kMaxDim) smax[tid] = 0u;
    }
    __syncthreads();

    int E = 0;
    float cap = 0.0f;
    if constexpr (FixedHist<HT>::value) {
      const float prev = st.hcap;
      if (!(prev > 0.0f)) {
        // first iteration: per dimension the largest weight factor
        // (positive floats order as their bit patterns)
        const T Nt = (T)N;
        for (int e = tid; e < dN; e += bs) {
          const T f = POW2 ? sC[e].span : Nt * sC[e].span;
          atomicMax(&smax[e / N], __float_as_uint((float)f));
        }
        __syncthreads();
      }
      if (tid == 0) {
        float cv;
        if (prev > 0.0f) {
          cv = prev;
        } else {
          float w = 1.0f, q = 1.0f;
          for (int j = 0; j < d; ++j) w = w * __uint_as_float(smax[j]);
          if (J.family == PRODUCT_PEAK) {
            for (int j = 0; j < d; ++j) q = q * (float)pp0[j];
            q = 1.0f / q;
          }
          const float v = w * q;
          cv = v * v;
        }
        // a cap that is not finite or too large for the sums' exponent range
        // (an integrand far above 1) sends every value to the FP64 histogram
        if (!(cv <= 0x1p100f)) cv = 0.0f;
        // 2^E >= 4 cnt c bounds the fixed-point total of every bin
        const double B = 4.0 * (double)cv * (double)(cnt > 0 ? cnt : 1);
        int ex = 0;
        (void)frexp(B, &ex);
        smax[kMaxDim] = (uint32_t)ex;
        smax[kMaxDim + 1] = __float_as_uint(cv);
      }
      __syncthreads();
      E = (int)smax[kMaxDim];
      cap = __uint_as_float(smax[kMaxDim + 1]);
    }
    double S1 = 0.0, S2 = 0.0;
    auto sample = [&](auto fam, auto rem) {
      sample_tile<T, HT, decltype(fam)::value, NB, ILP, POW2, decltype(rem)::value>(
          J, st.T, i0, cnt, sC, sH, pp0, pp1, E, cap, st.shift, sHx, S1, S2);
    };
#ifdef CCUBA_RTC
    sample(Int<USER>{}, Int<FULL ? 4 : 0>{});
#else
    auto sample_family = [&](auto rem) {
      switch (J.family) {
        case GAUSSIAN: sample(Int<GAUSSIAN>{}, rem); break;
        case OSCILLATORY: sample(Int<OSCILLATORY>{}, rem); break;
        case PRODUCT_PEAK: sample(Int<PRODUCT_PEAK>{}, rem); break;
        case CORNER_PEAK: sample(Int<CORNER_PEAK>{}, rem); break;
        default: sample(Int<C0>{}, rem); break;
      }
    };
    if constexpr (FULL) {
      sample_family(Int<4>{});
    } else {
      switch (d - 4 * (NB - 1)) {
        case 1: sample_family(Int<1>{}); break;
        case 2: sample_family(Int<2>{}); break;
        case 3: sample_family(Int<3>{}); break;
        default: sample_family(Int<4>{}); break;
      }
    }
#endif
    S1 = wave_sum(S1);
    S2 = wave_sum(S2);
    if (lane == 0) {
      red[0][wid] = S1;
      red[1][wid] = S2;
    }
    __syncthreads();
    if (tid == 0) {
      double a = 0.0, b = 0.0;
      for (int q = 0; q < (bs >> 6); ++q) {
        a += red[0][q];
        b += red[1][q];
      }
      J.tsums[2 * lt] = a;
      J.tsums[2 * lt + 1] = b;
    }
    double *th = J.thist + (long long)lt * dN;
    if constexpr (FixedHist<HT>::value && sizeof(T) == 8) {
      for (int e = tid; e < dN; e += bs)
        th[e] = ldexp((double)sH[dN + e], E - 59) + ldexp((double)sH[e], E - 91) + sHx[e];
    } else if constexpr (FixedHist<HT>::value) {
      for (int e = tid; e < dN; e += bs) th[e] = ldexp((double)sH[e], E - 62) + sHx[e];
    } else {
      for (int e = tid; e < dN; e += bs) th[e] = (double)sH[e];
    }

    __syncthreads();
  }
}

#ifndef CCUBA_RTC
// ---------------------------------------------------------------------------
// launchers of the instances of one (precision, histogram type)

template <typename T, typename HT, int ILP, int NB>
static void launch_dosample_cls(const VegasArgs &A, bool pow2, bool full, int grid, int block,
                                size_t lds, hipStream_t s) {
  if (pow2) {
    if (full)
      hipLaunchKernelGGL((vegas_dosample_kernel<T, HT, ILP, NB, true, true>), dim3(grid),
                         dim3(block), lds, s, A);
    else
      hipLaunchKernelGGL((vegas_dosample_kernel<T, HT, ILP, NB, true, false>), dim3(grid),
                         dim3(block), lds, s, A);
  } else {
    if (full)
      hipLaunchKernelGGL((vegas_dosample_kernel<T, HT, ILP, NB, false, true>), dim3(grid),
                         dim3(block), lds, s, A);
    else
      hipLaunchKernelGGL((vegas_dosample_kernel<T, HT, ILP, NB, false, false>), dim3(grid),
                         dim3(block), lds, s, A);
  }
}

template <typename T, typename HT, int ILP>
static void launch_dosample_ilp(const VegasArgs &A, int nb, bool pow2, bool full, int grid,
                                int block, size_t lds, hipStream_t s) {
  switch (nb) {
    case 1: launch_dosample_cls<T, HT, ILP, 1>(A, pow2, full, grid, block, lds, s); break;
    case 2: launch_dosample_cls<T, HT, ILP, 2>(A, pow2, full, grid, block, lds, s); break;
    case 3: launch_dosample_cls<T, HT, ILP, 3>(A, pow2, full, grid, block, lds, s); break;
    default: launch_dosample_cls<T, HT, ILP, 4>(A, pow2, full, grid, block, lds, s); break;
  }
}

template <typename T, typename HT>
static hipError_t launch_dosample_t(const VegasArgs &A, int nb, bool pow2, bool full, int grid,
                                    int block, size_t lds, hipStream_t s) {
  if (A.ilp == 2)
    launch_dosample_ilp<T, HT, 2>(A, nb, pow2, full, grid, block, lds, s);
  else
    launch_dosample_ilp<T, HT, 1>(A, nb, pow2, full, grid, block, lds, s);
  return hipGetLastError();
}

template <typename T, typename HT, int ILP, int NB>
static void dosample_fns_cls(std::vector<const void *> &fns) {
  fns.push_back((const void *)vegas_dosample_kernel<T, HT, ILP, NB, true, true>);
  fns.push_back((const void *)vegas_dosample_kernel<T, HT, ILP, NB, true, false>);
  fns.push_back((const void *)vegas_dosample_kernel<T, HT, ILP, NB, false, true>);
  fns.push_back((const void *)vegas_dosample_kernel<T, HT, ILP, NB, false, false>);
}

template <typename T, typename HT>
static void dosample_fns_t(std::vector<const void *> &fns) {
  dosample_fns_cls<T, HT, 1, 1>(fns);
  dosample_fns_cls<T, HT, 1, 2>(fns);
  dosample_fns_cls<T, HT, 1, 3>(fns);
  dosample_fns_cls<T, HT, 1, 4>(fns);
  dosample_fns_cls<T, HT, 2, 1>(fns);
  dosample_fns_cls<T, HT, 2, 2>(fns);
  dosample_fns_cls<T, HT, 2, 3>(fns);
  dosample_fns_cls<T, HT, 2, 4>(fns);
}

#endif  // CCUBA_RTC

}  // namespace ccuba
