// Bitonic sorting and merging of 64-bit keys held by one wave: key 64 q + lane is v[q] of the lane.
//
// Bound by the issue of a chain of dependent vector instructions, so every step is made short.
// Partners 64 keys or more apart are two registers of one lane.  Partners inside a row of 16 lanes
// are reached with data-parallel-primitive moves (quad permutations for 1 and 2 lanes, the row
// turned by 8, and for 4 lanes the row turned by 12 for the banks whose partner is above, by 4 for
// the others).  Partners 16 and 32 lanes away: one swap of half-rows or half-waves of a register
// with its copy leaves every lane with both keys of its pair, the lower position's first.  The side
// a lane keeps is a constant of the step, so it is folded into the compare's mask as a literal.
#pragma once

#include "ann_device.hpp"

namespace annmi {

template <u32 J>
__device__ __forceinline__ u32 lane_partner_word(u32 x) {
  static_assert(J == 1 || J == 2 || J == 4 || J == 8, "partners inside a row of 16 lanes");
  if constexpr (J == 1)
    return (u32)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true);
  else if constexpr (J == 2)
    return (u32)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true);
  else if constexpr (J == 4)
    return (u32)__builtin_amdgcn_update_dpp(__builtin_amdgcn_update_dpp(0, (int)x, 0x12C, 0xF, 0x5, false), (int)x, 0x124,
                                            0xF, 0xA, false);
  else
    return (u32)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, true);
}

// One compare-exchange between positions J apart, in runs of K positions of alternating direction
// (the first ascending, or descending with DESC), followed by the steps for J / 2, J / 4, ... 1.
template <int KPL, u32 K, u32 J, bool DESC>
struct BitonicStep {
  static constexpr bool ascending(u32 pos) { return ((pos & K) == 0) != DESC; }
  // bit l: lane l keeps the first of (its own key, its partner's) when that is the smaller
  static constexpr u64 keep_smaller(u32 q) {
    u64 m = 0;
    for (u32 l = 0; l < 64; ++l)
      if (((l & J) == 0) == ascending(64u * q + l)) m |= 1ull << l;
    return m;
  }
  template <u32 Q>
  static __device__ __forceinline__ void lanes(u64& v) {
    constexpr u64 keep = keep_smaller(Q);
    u64 x = v, y;
    if constexpr (J < 16) {
      y = ((u64)lane_partner_word<J>((u32)(v >> 32)) << 32) | lane_partner_word<J>((u32)v);
    } else {  // (x, y) = the keys of the pair's lower and upper position, the same in both lanes
      const u32 lo = (u32)v, hi = (u32)(v >> 32);
      if constexpr (J == 16) {
        const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        x = ((u64)h[0] << 32) | l[0];
        y = ((u64)h[1] << 32) | l[1];
      } else {
        const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        x = ((u64)h[0] << 32) | l[0];
        y = ((u64)h[1] << 32) | l[1];
      }
    }
    // (equal keys: either is right)
    if constexpr (KPL == 1) {
      v = __builtin_amdgcn_inverse_ballot_w64(ballot(x < y) ^ ~keep) ? x : y;
    } else {
      // a constant used for several registers would be moved to scalar registers of its own, and
      // held there all through the caller's loop: six more, and with them a wave per SIMD
      u32 lo = (u32)~keep, hi = (u32)(~keep >> 32);
      asm volatile("" : "+s"(lo));
      if constexpr ((u32)keep == (u32)(keep >> 32))
        hi = lo;
      else
        asm volatile("" : "+s"(hi));
      v = __builtin_amdgcn_inverse_ballot_w64(ballot(x < y) ^ (((u64)hi << 32) | lo)) ? x : y;
    }
  }
  template <u32 Q>
  static __device__ __forceinline__ void all_lanes(u64 (&v)[KPL]) {
    lanes<Q>(v[Q]);
    if constexpr (Q + 1 < (u32)KPL) all_lanes<Q + 1>(v);
  }
  static __device__ __forceinline__ void run(u64 (&v)[KPL]) {
    if constexpr (J >= 64) {
      constexpr u32 dq = J / 64;
#pragma unroll
      for (u32 q = 0; q < (u32)KPL; ++q) {
        if ((q & dq) == 0) {
          const u64 x = v[q], y = v[q | dq];
          const bool swap = (x > y) == ascending(64u * q);  // (K > J >= 64: the lane bits do not matter)
          v[q] = swap ? y : x;
          v[q | dq] = swap ? x : y;
        }
      }
    } else {
      all_lanes<0>(v);
    }
    if constexpr (J > 1) BitonicStep<KPL, K, J / 2, DESC>::run(v);
  }
};

// Sorts runs of KMAX positions (BitonicStage<KPL, 2, DESC, KMAX>; KMAX = 64 * KPL: all the keys); v
// must already be runs of K / 2 positions of alternating direction.
template <int KPL, u32 K, bool DESC, u32 KMAX = 64u * KPL>
struct BitonicStage {
  static __device__ __forceinline__ void run(u64 (&v)[KPL]) {
    BitonicStep<KPL, K, K / 2, DESC>::run(v);
    if constexpr (K < KMAX) BitonicStage<KPL, 2 * K, DESC, KMAX>::run(v);
  }
};

// Ascending order from a bitonic sequence.
template <int KPL>
__device__ __forceinline__ void bitonic_merge(u64 (&v)[KPL]) {
  BitonicStep<KPL, 64u * KPL, 32u * KPL, false>::run(v);
}

}  // namespace annmi
