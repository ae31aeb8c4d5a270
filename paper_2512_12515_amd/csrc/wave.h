// Wave-level sums of doubles (64 lanes) by DPP moves: a shuffle through the LDS crossbar takes
// about 60 cycles a step, a DPP move 8.
#pragma once

#include <hip/hip_runtime.h>

namespace pprpa {
namespace {

template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_move(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// The value of lane l (uniform).
__device__ __forceinline__ double lane_value(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Sum over the wave, in a fixed order (every lane gets it): running sums within the rows of 16
// lanes, then across the rows.
__device__ __forceinline__ double wave_total(double v) {
  v += dpp_move<0x111, 0xf>(v);  // row_shr:1
  v += dpp_move<0x112, 0xf>(v);  // row_shr:2
  v += dpp_move<0x114, 0xf>(v);  // row_shr:4
  v += dpp_move<0x118, 0xf>(v);  // row_shr:8
  v += dpp_move<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp_move<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
  return lane_value(v, 63);
}

// 1 / x to a rounding or two (hardware reciprocal, two Newton steps): for recurrences where an IEEE
// division's dependent chain is three times as long. x normal and not zero.
__device__ __forceinline__ double fast_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
  return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

}  // namespace
}  // namespace pprpa
