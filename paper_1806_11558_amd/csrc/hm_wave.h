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

// Sums of N = 4 or 8 values over the wavefront together: every step halves the
// values by handing each half of the lanes one value of a pair, first between
// the halves and quarters of the wavefront by lane swaps (three instructions
// per pair), then within rows of 16 lanes.  The sum of value k is in lane
// k * 64 / N, in a fixed order; 34 instructions for eight values where eight
// wsum take 144.
__device__ inline double swap_add32(double a, double b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a);
  const unsigned long long y = (unsigned long long)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  return __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
         __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ inline double swap_add16(double a, double b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a);
  const unsigned long long y = (unsigned long long)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  return __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
         __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ inline double swap_add8(double a, double b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a);
  const unsigned long long y = (unsigned long long)__double_as_longlong(b);
  int r[2], k[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int u = (int)(unsigned)(x >> (32 * h)), v = (int)(unsigned)(y >> (32 * h));
    r[h] = __builtin_amdgcn_update_dpp(0, u, 0x128, 0xF, 0x3, false);      // row_ror:8
    r[h] = __builtin_amdgcn_update_dpp(r[h], v, 0x128, 0xF, 0xC, false);
    k[h] = __builtin_amdgcn_update_dpp(u, v, 0xE4, 0xF, 0xC, false);       // lanes 8..15: v
  }
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)k[1] << 32) | (unsigned)k[0])) +
         __longlong_as_double((long long)(((unsigned long long)(unsigned)r[1] << 32) | (unsigned)r[0]));
}
__device__ inline double wsums(const double (&p)[4]) {
  return rowsum(swap_add16(swap_add32(p[0], p[2]), swap_add32(p[1], p[3])));
}
__device__ inline double wsums(const double (&p)[8]) {
  const double a = swap_add16(swap_add32(p[0], p[4]), swap_add32(p[2], p[6]));
  const double b = swap_add16(swap_add32(p[1], p[5]), swap_add32(p[3], p[7]));
  double v = swap_add8(a, b);
  v += dpp_v<0xB1, 0xF>(v);
  v += dpp_v<0x4E, 0xF>(v);
  v += dpp_v<0x141, 0xF>(v);
  return v;
}

// Orders a wavefront's own memory accesses: what its lanes wrote before, all
// of them read after (no instruction: a wavefront's accesses go in order).
__device__ inline void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace hm
