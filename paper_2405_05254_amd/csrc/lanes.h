// Reductions across the lanes of a wavefront that stay in registers (DPP within a row of 16 lanes, gfx950's row swaps between
// rows). A shuffle goes through the LDS crossbar: a hundred clocks each, one behind the other, at the end of every kernel
// here that is over in a few microseconds (a token step of 43 launches took 12 us less without those of its
// matrix-vector products). Every lane ends with the result, and all lanes with the same bits.
#pragma once
#include <hip/hip_runtime.h>

namespace yoco {

struct LaneSum {
  static __device__ __forceinline__ float of(float a, float b) { return a + b; }
};
struct LaneMax {
  static __device__ __forceinline__ float of(float a, float b) { return fmaxf(a, b); }
};
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
// with lane ^ 16
template <typename F>
__device__ __forceinline__ float with_next_row(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return F::of(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// with lane ^ 32
template <typename F>
__device__ __forceinline__ float with_other_half(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return F::of(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// over 4 and 16 consecutive lanes, nearest first
template <typename F>
__device__ __forceinline__ float over4(float x) {
  x = F::of(x, dpp_mov<0xB1>(x));           // quad_perm [1,0,3,2]
  return F::of(x, dpp_mov<0x4E>(x));        // quad_perm [2,3,0,1]
}
template <typename F>
__device__ __forceinline__ float over16(float x) {
  x = over4<F>(x);
  x = F::of(x, dpp_mov<0x141>(x));          // row_half_mirror: the other quad
  return F::of(x, dpp_mov<0x140>(x));       // row_mirror: the other eight
}
// over 8 consecutive lanes, farthest first
template <typename F>
__device__ __forceinline__ float over8(float x) {
  const int u = __float_as_int(x);
  const int below = __builtin_amdgcn_update_dpp(u, u, 0x104, 0xf, 0x5, false);      // row_shl:4 into the first and third quad of a row
  x = F::of(x, __int_as_float(__builtin_amdgcn_update_dpp(below, u, 0x114, 0xf, 0xa, false)));   // row_shr:4 into the others
  x = F::of(x, dpp_mov<0x4E>(x));
  return F::of(x, dpp_mov<0xB1>(x));
}
// over the four lanes that share lane % 16
template <typename F>
__device__ __forceinline__ float over_rows(float x) { return with_other_half<F>(with_next_row<F>(x)); }
// over 32 and 64, farthest first: the order of a butterfly of shuffles
template <typename F>
__device__ __forceinline__ float over32(float x) {
  x = with_next_row<F>(x);
  return over8<F>(F::of(x, dpp_mov<0x128>(x)));     // row_ror:8
}
template <typename F>
__device__ __forceinline__ float over64(float x) { return over32<F>(with_other_half<F>(x)); }
// over64 of x[0] + of x[1], of four (x[0] + x[1]) + (x[2] + x[3]), with the same bits: behind the first exchanges a row of lanes has
// one of them to itself, so that the others run together.
template <int N>
__device__ __forceinline__ float sum_over64(const float (&x)[N]) {
  static_assert(N == 2 || N == 4, "a half or a row of lanes for each");
  float half[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[i]), __float_as_uint(x[i + N - 2]), false, false);
    half[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(half[0]), __float_as_uint(half[1]), false, false);
  float row = __uint_as_float(r[0]) + __uint_as_float(r[1]);                  // row i: x[i % N]
  row = with_next_row<LaneSum>(over8<LaneSum>(row + dpp_mov<0x128>(row)));    // row_ror:8
  return N == 2 ? row : with_other_half<LaneSum>(row);
}

}  // namespace yoco
