// Sums over a wave64 by data-parallel-primitive moves (lane shifts within the vector ALU; the
// LDS-based shuffles take about ten times as long per step, and a kernel that sums at its head
// or tail waits for six of them).
#pragma once

#include <hip/hip_runtime.h>

namespace sfem {

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_moved(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, ROW_MASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROW_MASK, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Value of v in lane `lane`, in every lane (lane uniform).
__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum over the lanes 0 .. last of the wave, in every lane; lanes beyond last may not exist.
// Inclusive prefix sums within the rows of 16 lanes (shifts by 1, 2, 4, 8), then the last lane
// of a row added to the rows after it: a fixed order.
__device__ __forceinline__ double wave_total(double v, int last = 63) {
  v += dpp_moved<0x111, 0xf>(v);
  v += dpp_moved<0x112, 0xf>(v);
  v += dpp_moved<0x114, 0xf>(v);
  v += dpp_moved<0x118, 0xf>(v);
  v += dpp_moved<0x142, 0xa>(v);  // lane 15 -> row 1, lane 47 -> row 3
  v += dpp_moved<0x143, 0xc>(v);  // lane 31 -> rows 2 and 3
  return lane_value(v, last);
}

}  // namespace sfem
