// Exchanges between the lanes of a wave.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace netsim_dev {

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_min(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = (int)b, hi = (int)(b >> 32);
  const int l2 = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xF, false);
  const int h2 = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xF, false);
  const double w = __longlong_as_double(((long long)h2 << 32) | (unsigned)l2);
  return w < v ? w : v;
}

// Minimum over the 64 lanes, the same value in every lane (no shared memory:
// exchanges inside rows of 16 lanes, then row 0 -> 1 and 2 -> 3, then the
// lower half to the upper one; lane 63 holds the result).
__device__ __forceinline__ double wmin(double v) {
  v = dpp_min<0xB1, 0xF>(v);   // lanes 1 apart
  v = dpp_min<0x4E, 0xF>(v);   // 2 apart
  v = dpp_min<0x141, 0xF>(v);  // mirrored in half rows
  v = dpp_min<0x140, 0xF>(v);  // mirrored in rows
  v = dpp_min<0x142, 0xA>(v);  // lane 15 of the row before, rows 1 and 3
  v = dpp_min<0x143, 0xC>(v);  // lane 31, rows 2 and 3
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, 63);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Position of this lane among the lanes set in mask.
__device__ __forceinline__ int rank_in(uint64_t mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

}  // namespace netsim_dev
