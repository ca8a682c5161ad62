// wave.h -- wavefront reductions by DPP (no LDS traffic).
#pragma once
#include <hip/hip_runtime.h>

namespace ccuba {

// One DPP step: the value of the lane the control selects, `identity' in
// lanes without a source.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or(double v, double identity) {
  const long long b = __double_as_longlong(v), z = __double_as_longlong(identity);
  const int lo = __builtin_amdgcn_update_dpp((int)z, (int)b, CTRL, ROWS, 0xf, false);
  const int hi =
      __builtin_amdgcn_update_dpp((int)(z >> 32), (int)(b >> 32), CTRL, ROWS, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// A reduction over the wavefront, its result in lane 63: the row shifts leave
// each row's result in its lane 15, the row broadcasts carry it on.
template <typename OP>
__device__ __forceinline__ double wave_reduce63(double v, double identity, OP op) {
  v = op(v, dpp_or<0x111, 0xf>(v, identity));  // row_shr:1
  v = op(v, dpp_or<0x112, 0xf>(v, identity));  // row_shr:2
  v = op(v, dpp_or<0x114, 0xf>(v, identity));  // row_shr:4
  v = op(v, dpp_or<0x118, 0xf>(v, identity));  // row_shr:8
  v = op(v, dpp_or<0x142, 0xa>(v, identity));  // row_bcast:15 into rows 1 and 3
  v = op(v, dpp_or<0x143, 0xc>(v, identity));  // row_bcast:31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ double wave_reduce63_sum(double v) {
  return wave_reduce63(v, 0.0, [](double a, double b) { return a + b; });
}

}  // namespace ccuba
