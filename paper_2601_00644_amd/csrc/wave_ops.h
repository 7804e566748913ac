// Exchanges between the lanes of a wave without LDS (gfx950): data-parallel moves within rows of 16 lanes, row and half swaps beyond.
// An exchange through LDS (__shfl_xor) is a round trip to LDS, and the kernels whose launches are short chains of dependent
// steps go through a dozen of them; these take a few cycles.  The sums they form are the same, in the same order.  One fp32 request
// through two layers 66.8 -> 60.7 us, one 1B request on 16 layers 744 -> 738, sampling from 152064 bf16 logits 54.4 -> 53.3.
// All lanes of the rows (1 .. 8) or of the wave (16, 32) that take part must be active.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

template <int OFF>
__device__ __forceinline__ uint32_t lane_xor_bits(uint32_t x) {
  static_assert(OFF == 1 || OFF == 2 || OFF == 4 || OFF == 8 || OFF == 16 || OFF == 32, "");
  if constexpr (OFF == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true);         // quad_perm 1 0 3 2
  else if constexpr (OFF == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true);    // quad_perm 2 3 0 1
  else if constexpr (OFF == 4) {   // row_shl 4 into quads 0 and 2, row_shr 4 into quads 1 and 3
    const int t = __builtin_amdgcn_update_dpp(0, (int)x, 0x104, 0xF, 0x5, false);
    return (uint32_t)__builtin_amdgcn_update_dpp(t, (int)x, 0x114, 0xF, 0xA, false);
  } else if constexpr (OFF == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, true);   // row_ror 8
  else {
    const bool upper = (__lane_id() & OFF) != 0;
    if constexpr (OFF == 16) {
      const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
      return upper ? r[0] : r[1];
    } else {
      const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
      return upper ? r[0] : r[1];
    }
  }
}

// The value of lane l ^ OFF.
template <int OFF, typename T>
__device__ __forceinline__ T lane_xor(T v) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "");
  if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, lane_xor_bits<OFF>(__builtin_bit_cast(uint32_t, v)));
  else {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = lane_xor_bits<OFF>((uint32_t)b), hi = lane_xor_bits<OFF>((uint32_t)(b >> 32));
    return __builtin_bit_cast(T, (uint64_t)lo | ((uint64_t)hi << 32));
  }
}

// lo of the lanes without the bit OFF and hi of those with it, each added to its partner's: what lane l keeps is lo or hi.
template <int OFF>
__device__ __forceinline__ float lane_fold(float lo, float hi, int lane) {
  if constexpr (OFF == 16 || OFF == 32) {   // the swap leaves own and partner's value of the kept one in the two registers
    const uint32_t a = __builtin_bit_cast(uint32_t, lo), b = __builtin_bit_cast(uint32_t, hi);
    if constexpr (OFF == 16) {
      const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
      return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
    } else {
      const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
      return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
    }
  } else {
    const float send = (lane & OFF) ? lo : hi, keep = (lane & OFF) ? hi : lo;
    return keep + lane_xor<OFF>(send);
  }
}
template <int OFF>
__device__ __forceinline__ float lane_pair_sum(float v) {
  if constexpr (OFF == 16 || OFF == 32) return lane_fold<OFF>(v, v, 0);
  else return v + lane_xor<OFF>(v);
}

// f(an integral constant) for the offsets FROM, FROM / 2, .. 1.
template <int FROM, typename F>
__device__ __forceinline__ void lane_steps(F &&f) {
  f(std::integral_constant<int, FROM>{});
  if constexpr (FROM > 1) lane_steps<FROM / 2>(f);
}

// Sum, maximum and (maximum, lowest index that attains it) over groups of 2 FROM lanes, in every lane of the group.
template <int FROM = 32, typename T>
__device__ __forceinline__ T lanes_sum(T v) {
  lane_steps<FROM>([&](auto off) { v += lane_xor<decltype(off)::value>(v); });
  return v;
}
template <int FROM = 32>
__device__ __forceinline__ float lanes_max(float v) {
  lane_steps<FROM>([&](auto off) { v = fmaxf(v, lane_xor<decltype(off)::value>(v)); });
  return v;
}
template <int FROM = 32>
__device__ __forceinline__ void lanes_argmax(float &mx, int &ai) {
  lane_steps<FROM>([&](auto off) {
    const float om = lane_xor<decltype(off)::value>(mx);
    const int oi = lane_xor<decltype(off)::value>(ai);
    if (om > mx || (om == mx && oi < ai)) { mx = om; ai = oi; }
  });
}
__device__ __forceinline__ float wave_sum(float v) {
  lane_steps<32>([&](auto off) { v = lane_pair_sum<decltype(off)::value>(v); });
  return v;
}
