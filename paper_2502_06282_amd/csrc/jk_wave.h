// Reductions over a wave of 64 lanes in registers: exchanges between lanes by DPP and lane swaps cost a few cycles each,
// where a shuffle is a round trip through LDS.  Not installed.
#pragma once
#include <hip/hip_runtime.h>

namespace jk {
namespace dev {

// The result is in every lane: exchanges with lane ^ 1, ^ 2 (quad_perm), then, the halves being uniform by then, mirrored
// within 8 and 16, then halves of 32 and of 64 swapped.
template <int CTRL>
__device__ __forceinline__ int dpp(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp64(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)dpp<CTRL>((int)b), hi = (unsigned)dpp<CTRL>((int)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
typedef unsigned wave_u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned other16(unsigned v, bool upper) {  // the value of lane ^ 16
  const wave_u32x2 s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return upper ? s[0] : s[1];
}
__device__ __forceinline__ unsigned other32(unsigned v, bool upper) {  // the value of lane ^ 32
  const wave_u32x2 s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return upper ? s[0] : s[1];
}
__device__ __forceinline__ double swap64(double v, bool by32) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const int lane = __lane_id();
  unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
  if (by32) {
    lo = other32(lo, lane & 32);
    hi = other32(hi, lane & 32);
  } else {
    lo = other16(lo, lane & 16);
    hi = other16(hi, lane & 16);
  }
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp64<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp64<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp64<0x141>(v);  // row_half_mirror
  v += dpp64<0x140>(v);  // row_mirror
  v += swap64(v, false);
  v += swap64(v, true);
  return v;
}
// 2^(d (hi + lo)) for d <= 0: the whole part of the exponent apart, the rest of it exact to the last place but one product's rounding, so
// that what the instruction itself rounds is all there is
__device__ __forceinline__ float exp_scaled(float d, float hi, float lo) {
  const float n = __builtin_rintf(fmaxf(d * hi, -300.f));
  const float e = __builtin_ldexpf(__builtin_amdgcn_exp2f(fmaf(d, lo, fmaf(d, hi, -n))), (int)n);
  return d == -INFINITY ? 0.f : e;
}
// Over the 32 lanes of each half of a wave, in all of them
__device__ __forceinline__ float half_max(float v) {
  v = fmaxf(v, __int_as_float(dpp<0xB1>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp<0x4E>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp<0x141>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp<0x140>(__float_as_int(v))));
  return fmaxf(v, __uint_as_float(other16(__float_as_uint(v), __lane_id() & 16)));
}
__device__ __forceinline__ float half_sum(float v) {
  v += __int_as_float(dpp<0xB1>(__float_as_int(v)));
  v += __int_as_float(dpp<0x4E>(__float_as_int(v)));
  v += __int_as_float(dpp<0x141>(__float_as_int(v)));
  v += __int_as_float(dpp<0x140>(__float_as_int(v)));
  return v + __uint_as_float(other16(__float_as_uint(v), __lane_id() & 16));
}
// Inclusive sums over the lanes: rows of 16 by shifts, then the rows' totals broadcast into the rows behind them
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, __int_as_float(dpp<0xB1>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp<0x4E>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp<0x141>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp<0x140>(__float_as_int(v))));
  const int lane = __lane_id();
  v = fmaxf(v, __uint_as_float(other16(__float_as_uint(v), lane & 16)));
  v = fmaxf(v, __uint_as_float(other32(__float_as_uint(v), lane & 32)));
  return v;
}
__device__ __forceinline__ int wave_min(int v) {
  v = min(v, dpp<0xB1>(v));
  v = min(v, dpp<0x4E>(v));
  v = min(v, dpp<0x141>(v));
  v = min(v, dpp<0x140>(v));
  const int lane = __lane_id();
  v = min(v, (int)other16((unsigned)v, lane & 16));
  v = min(v, (int)other32((unsigned)v, lane & 32));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
  v += __int_as_float(dpp<0xB1>(__float_as_int(v)));
  v += __int_as_float(dpp<0x4E>(__float_as_int(v)));
  v += __int_as_float(dpp<0x141>(__float_as_int(v)));
  v += __int_as_float(dpp<0x140>(__float_as_int(v)));
  const int lane = __lane_id();
  v += __uint_as_float(other16(__float_as_uint(v), lane & 16));
  v += __uint_as_float(other32(__float_as_uint(v), lane & 32));
  return v;
}

}  // namespace dev
}  // namespace jk
