// Exchanges between the lanes of a wavefront on the vector unit.  __shfl_xor goes through the LDS crossbar, some 60 clocks for each
// 32 bits and step of a chain; within 16 lanes DPP reads another lane's register as an operand, and gfx950 swaps 16- and 32-lane rows in
// one instruction.  Rounds of the tiny fp32 pair (10 rows, 75 launches) 349 -> 304 us with these and the loads its linear layers want last
// requested first, a verification of one sequence 18.1 -> 16.5, 24-row rounds of the 1B shape 4969 -> 4898.  The butterflies below take the
// partners that __shfl_xor(v, o) takes, o from FROM to LAST, halved or doubled from step to step: in the same order, the same bits.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ssd {

// What a lane and its partner (lane ^ O) hold of `v`: operands of an operation that gives both the same result whichever comes first (for a
// choice between two values that means no NaN among them).
template <int O>
__device__ __forceinline__ void lane_pair(uint32_t v, uint32_t& a, uint32_t& b) {
  static_assert(O == 1 || O == 2 || O == 4 || O == 8 || O == 16 || O == 32, "a bit of the lane index");
  if constexpr (O == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    a = r[0];
    b = r[1];
  } else if constexpr (O == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    a = r[0];
    b = r[1];
  } else {
    a = v;
    if constexpr (O == 8) b = __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, false);        // row rotated by 8
    if constexpr (O == 4) {
      const uint32_t m = __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, false);             // 8 lanes mirrored (lane ^ 7)
      b = __builtin_amdgcn_update_dpp(0, m, 0x1b, 0xf, 0xf, false);                             // and back within four (lane ^ 3)
    }
    if constexpr (O == 2) b = __builtin_amdgcn_update_dpp(0, v, 0x4e, 0xf, 0xf, false);
    if constexpr (O == 1) b = __builtin_amdgcn_update_dpp(0, v, 0xb1, 0xf, 0xf, false);
  }
}

// op over lanes FROM apart, then half (or, LAST > FROM, twice) as far at each step until LAST apart: a whole wavefront is 32 to 1.  op has
// to be commutative.  Every lane gets its group's result.  A sum's bits depend on the order: the narrow pass's row scales and the sums
// over rows of 16 lanes take their nearest lanes first.
template <int FROM = 32, int LAST = 1, typename T, typename Op>
__device__ __forceinline__ T lanes_reduce(T v, Op op) {
  static_assert(sizeof(T) % 4 == 0, "whole registers");
  struct Words { uint32_t w[sizeof(T) / 4]; };
  const Words x = __builtin_bit_cast(Words, v);
  Words a, b;
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 4; ++i) lane_pair<FROM>(x.w[i], a.w[i], b.w[i]);
  const T r = op(__builtin_bit_cast(T, a), __builtin_bit_cast(T, b));
  if constexpr (FROM > LAST) return lanes_reduce<FROM / 2, LAST>(r, op);
  else if constexpr (FROM < LAST) return lanes_reduce<FROM * 2, LAST>(r, op);
  else return r;
}
template <int FROM = 32, int LAST = 1, typename T>
__device__ __forceinline__ T lanes_sum(T v) {
  return lanes_reduce<FROM, LAST>(v, [](T a, T b) { return a + b; });
}
template <int FROM = 32, int LAST = 1>
__device__ __forceinline__ float lanes_max(float v) {
  return lanes_reduce<FROM, LAST>(v, [](float a, float b) { return fmaxf(a, b); });
}

// Half of the lanes keep `lo` and hand over `hi`, the others (those with bit O of their index set) the reverse: every lane's own value
// plus what it is handed.
template <int O>
__device__ __forceinline__ float lanes_split_sum(float lo, float hi) {
  if constexpr (O == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  } else if constexpr (O == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  } else {
    const bool up = (threadIdx.x & O) != 0;
    uint32_t own, other;
    lane_pair<O>(__float_as_uint(up ? lo : hi), own, other);
    return (up ? hi : lo) + __uint_as_float(other);
  }
}

}  // namespace ssd
