// Wavefront sums and broadcasts by DPP moves, shared by the setup and the
// solver kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace hm {

// ---- wavefront primitives (gfx9 DPP).  The row-of-16 butterfly (quad
// permutes, half mirror, mirror) followed by the two row broadcasts leaves
// the full result in lane 63; readlane makes it uniform.  Masked rows of a
// DPP move read 0.
template <int CTRL, int ROWMASK>
__device__ inline int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWMASK, 0xF, false);
}
__device__ inline int rdl_i(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
template <int C, int RM>
__device__ inline float dpp_v(float v) {
  return __int_as_float(dpp_i<C, RM>(__float_as_int(v)));
}
template <int C, int RM>
__device__ inline double dpp_v(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)dpp_i<C, RM>((int)(unsigned)b);
  const unsigned hi = (unsigned)dpp_i<C, RM>((int)(unsigned)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ inline float rdl_v(float v, int l) { return __int_as_float(rdl_i(__float_as_int(v), l)); }
__device__ inline double rdl_v(double v, int l) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)rdl_i((int)(unsigned)b, l);
  const unsigned hi = (unsigned)rdl_i((int)(unsigned)(b >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Sum over each row of 16 lanes, in every lane of the row, fixed order.
template <typename A>
__device__ inline A rowsum(A v) {
  v += dpp_v<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]
  v += dpp_v<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]
  v += dpp_v<0x141, 0xF>(v);   // row_half_mirror
  v += dpp_v<0x140, 0xF>(v);   // row_mirror
  return v;
}

// Sum over the wavefront, uniform result, fixed order.
template <typename A>
__device__ inline A wsum(A v) {
  v = rowsum(v);
  v += dpp_v<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp_v<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
  return rdl_v(v, 63);
}

// Orders a wavefront's own memory accesses: what its lanes wrote before, all
// of them read after (no instruction: a wavefront's accesses go in order).
__device__ inline void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace hm

