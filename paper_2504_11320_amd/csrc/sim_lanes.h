// sim_lanes.h -- lane-group operations of the kernels that run a replica on a
// group of G lanes (G a power of two; 64 / G groups in a wavefront): sums,
// minima and orders over a group with DPP lane permutations on the ALU.
#pragma once

#include "sim_common.h"

namespace wsim {
namespace {

// ---------------------------------------------------------- group lanes --
// DPP lane permutations inside 16-lane rows (gfx9 encodings): swap neighbours
// (quad_perm [1,0,3,2]), swap pairs (quad_perm [2,3,0,1]), mirror each half
// row (lane i <-> 7-i), mirror the row (i <-> 15-i).  After the first two a
// lane holds its quad's reduction; the half-row mirror pairs each lane with
// one of the other quad of its 8, the row mirror with one of the other 8 of
// its 16: an all-reduce over groups of 4, 8 or 16 aligned lanes that reads
// no lane outside the group.
constexpr int kDppSwap1 = 0xB1;
constexpr int kDppSwap2 = 0x4E;
constexpr int kDppHalfMirror = 0x141;
constexpr int kDppMirror = 0x140;

template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ uint64_t dpp64(uint64_t v) {
  return ((uint64_t)dpp32<CTRL>((uint32_t)(v >> 32)) << 32) | dpp32<CTRL>((uint32_t)v);
}

// Shift by one lane inside the 16-lane rows: row_shl:1 (lane i takes lane
// i+1) and row_shr:1 (lane i takes lane i-1); a row's end lane keeps 0.
constexpr int kDppShl1 = 0x101;
constexpr int kDppShr1 = 0x111;

// Groups of 32 or 64 lanes combine the 16-lane rows with lane-index XOR
// exchanges (16, then 32).
template <int MASK>
__device__ __forceinline__ uint32_t xor32(uint32_t v) {
  return (uint32_t)__shfl_xor((int)v, MASK, 64);
}
template <int MASK>
__device__ __forceinline__ uint64_t xor64(uint64_t v) {
  return ((uint64_t)xor32<MASK>((uint32_t)(v >> 32)) << 32) | xor32<MASK>((uint32_t)v);
}

template <int G, typename Op>
__device__ __forceinline__ uint64_t group_reduce64(uint64_t v, Op op) {
  if constexpr (G >= 2) v = op(v, dpp64<kDppSwap1>(v));
  if constexpr (G >= 4) v = op(v, dpp64<kDppSwap2>(v));
  if constexpr (G >= 8) v = op(v, dpp64<kDppHalfMirror>(v));
  if constexpr (G >= 16) v = op(v, dpp64<kDppMirror>(v));
  if constexpr (G >= 32) v = op(v, xor64<16>(v));
  if constexpr (G >= 64) v = op(v, xor64<32>(v));
  return v;
}
template <int G>
__device__ __forceinline__ int64_t group_sum(int64_t v) {
  return (int64_t)group_reduce64<G>((uint64_t)v, [](uint64_t a, uint64_t b) { return a + b; });
}
template <int G, typename Op>
__device__ __forceinline__ uint32_t group_reduce32(uint32_t v, Op op) {
  if constexpr (G >= 2) v = op(v, dpp32<kDppSwap1>(v));
  if constexpr (G >= 4) v = op(v, dpp32<kDppSwap2>(v));
  if constexpr (G >= 8) v = op(v, dpp32<kDppHalfMirror>(v));
  if constexpr (G >= 16) v = op(v, dpp32<kDppMirror>(v));
  if constexpr (G >= 32) v = op(v, xor32<16>(v));
  if constexpr (G >= 64) v = op(v, xor32<32>(v));
  return v;
}
// Sum of values whose group total fits in 32 bits (per-batch memory changes
// and counts).
template <int G>
__device__ __forceinline__ int32_t group_sum32(int32_t v) {
  return (int32_t)group_reduce32<G>((uint32_t)v, [](uint32_t a, uint32_t b) { return a + b; });
}
template <int G>
__device__ __forceinline__ uint32_t group_or(uint32_t v) {
  return group_reduce32<G>(v, [](uint32_t a, uint32_t b) { return a | b; });
}
// Minimum of two numbers (never NaN): one instruction, without the quieting
// of signalling NaNs that fmin asks for.  The wait states a DPP read of the
// result needs are part of it (the compiler adds none after inline asm).
__device__ __forceinline__ double min_f64(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2\n\ts_nop 1" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
template <int G>
__device__ __forceinline__ double group_min(double v) {
  const uint64_t r = group_reduce64<G>((uint64_t)__double_as_longlong(v), [](uint64_t a, uint64_t b) {
    return (uint64_t)__double_as_longlong(
        min_f64(__longlong_as_double((long long)a), __longlong_as_double((long long)b)));
  });
  return __longlong_as_double((long long)r);
}
// The value of segment lane k+1 (seg_next) or k-1 (seg_prev) of the group;
// the group's end lanes get values they do not use.
template <int G>
__device__ __forceinline__ uint32_t seg_next(uint32_t v) {
  if constexpr (G <= 16)
    return dpp32<kDppShl1>(v);
  else
    return (uint32_t)__shfl_down((int)v, 1u, G);
}
template <int G>
__device__ __forceinline__ uint32_t seg_prev(uint32_t v) {
  if constexpr (G <= 16)
    return dpp32<kDppShr1>(v);
  else
    return (uint32_t)__shfl_up((int)v, 1u, G);
}
template <int G>
__device__ __forceinline__ uint64_t seg_prev64(uint64_t v) {
  return ((uint64_t)seg_prev<G>((uint32_t)(v >> 32)) << 32) | seg_prev<G>((uint32_t)v);
}

// Conditions as lane masks in scalar registers: ballot of a plain comparison
// is the comparison alone, masks combine on the scalar unit, and in(mask) is
// the condition again.  (A ballot of a combined condition would take two more
// vector instructions, and HIP's __ballot and __any always do.)
using Mask = uint64_t;
__device__ __forceinline__ Mask ballot(bool pred) { return __builtin_amdgcn_ballot_w64(pred); }
__device__ __forceinline__ bool in(Mask m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Bits 0, G, 2G, ...: the first lanes of the groups.
template <int G>
__device__ constexpr Mask group_leaders() {
  Mask m = 0;
  for (int i = 0; i < 64; i += G) m |= 1ull << i;
  return m;
}
// This lane's group, and the lanes of it below this one.  With these two
// kept per lane a question about a group of a mask is three vector
// instructions; on the scalar unit it would be a chain of shifts.
template <int G>
__device__ __forceinline__ Mask group_of_lane() {
  return (G == 64 ? ~0ull : (1ull << (G & 63)) - 1ull) << (threadIdx.x & (64 - G));
}
template <int G>
__device__ __forceinline__ Mask below_lane() {
  return group_of_lane<G>() & ((1ull << threadIdx.x) - 1ull);
}
// (Every lane of the wavefront takes part in these.)
// All lanes of the groups that have a lane in m.
template <int G>
__device__ __forceinline__ Mask group_spread(Mask m) {
  if constexpr (G == 1) return m;
  return ballot((m & group_of_lane<G>()) != 0);
}
// The lowest and the highest lane of m in every group.
template <int G>
__device__ __forceinline__ Mask group_lowest(Mask m) {
  if constexpr (G == 1) return m;
  return m & ballot((m & below_lane<G>()) == 0);
}
template <int G>
__device__ __forceinline__ Mask group_highest(Mask m) {
  if constexpr (G == 1) return m;
  const Mask above = group_of_lane<G>() & ~((2ull << threadIdx.x) - 1ull);
  return m & ballot((m & above) == 0);
}
// Lanes with one of m at or below them in their group.
template <int G>
__device__ __forceinline__ Mask group_fill_up(Mask m) {
  if constexpr (G == 1) return m;
  return ballot((m & group_of_lane<G>() & ((2ull << threadIdx.x) - 1ull)) != 0);
}

// The group's G bits of a wavefront ballot (bit g = group lane g).
template <int G>
__device__ __forceinline__ uint64_t group_bits(bool pred) {
  const uint64_t b = ballot(pred);
  if constexpr (G == 64) {
    return b;
  } else {
    return (b >> (threadIdx.x & (64 - G))) & ((1ull << G) - 1ull);
  }
}

// Sum of v over the higher lanes of the group (lane index gl).
template <int G>
__device__ __forceinline__ int32_t sum_above(int32_t v, int gl) {
  constexpr int W = G < 16 ? G : 16;  // inside the 16-lane rows first
  const int x = gl & (W - 1);
  int32_t s = v;
  auto step = [&](int d, uint32_t up) __attribute__((always_inline)) {
    s += x + d < W ? (int32_t)up : 0;
  };
  // row_shl:d (0x100 + d): lane i takes lane i + d of its row
  if constexpr (G >= 2) step(1, dpp32<0x101>((uint32_t)s));
  if constexpr (G >= 4) step(2, dpp32<0x102>((uint32_t)s));
  if constexpr (G >= 8) step(4, dpp32<0x104>((uint32_t)s));
  if constexpr (G >= 16) step(8, dpp32<0x108>((uint32_t)s));
  if constexpr (G >= 32) {  // then the totals of the higher rows (their lane 0)
    const int base = (int)(threadIdx.x & (64 - G));
    const int32_t rows = s;
#pragma unroll
    for (int b = 16; b < G; b += 16) {
      const int32_t tot = __shfl(rows, base + b, 64);
      s += b > gl ? tot : 0;
    }
  }
  return s - v;
}

// lat_sum plus each group lane's v in lane order; `who`: ballot of the lanes
// whose v is not zero (the others' zeros leave the sum as it is).
template <int G>
__device__ __forceinline__ double add_in_order(double sum, double v, uint64_t who) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  auto from = [](uint64_t x) __attribute__((always_inline)) { return __longlong_as_double((long long)x); };
  if constexpr (G == 1) {
    return sum + v;
  } else if constexpr (G == 2) {
    sum += from(dpp64<0xA0>(b));
    return sum + from(dpp64<0xF5>(b));
  } else if constexpr (G == 4) {  // quad_perm [j,j,j,j]
    sum += from(dpp64<0x00>(b));
    sum += from(dpp64<0x55>(b));
    sum += from(dpp64<0xAA>(b));
    return sum + from(dpp64<0xFF>(b));
  } else {
    const int base = (int)(threadIdx.x & (64 - G));
    uint64_t some = who;  // lane j of any group, at bit j
    if constexpr (G <= 32) some |= some >> 32;
    if constexpr (G <= 16) some |= some >> 16;
    if constexpr (G <= 8) some |= some >> 8;
    if constexpr (G < 64) some &= (1ull << (G < 64 ? G : 0)) - 1ull;
    while (some != 0) {  // wavefront-uniform
      const int j = __builtin_ctzll(some);
      some &= some - 1ull;
      sum += __shfl(v, base + j, 64);
    }
    return sum;
  }
}

}  // namespace
}  // namespace wsim
