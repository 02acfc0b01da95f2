// skim_wave.h -- cross-lane moves of a 64-lane wave on the vector unit.
//
// __shfl_xor goes through the LDS permute unit (one such unit per CU, tens of
// cycles of latency).  The moves a butterfly needs exist on the vector unit:
// DPP quad permutes, half-row and row mirrors and a row rotation inside 16
// lanes, and gfx950's permlane16/32 swaps across rows.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace skim {

// LDS written by some lanes of a wave, then read by others of it: in program order
// for the compiler too.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int kCtrl> __device__ __forceinline__ uint32_t dpp_move(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, kCtrl, 0xF, 0xF, true);
}

// The two results of a row swap of x with itself: lanes of the lower row of
// a pair find their partner's value in `b`, lanes of the upper row in `a`;
// either way {a, b} = {own, partner}.
struct LanePair {
    uint32_t a, b;
};
__device__ __forceinline__ LanePair swap_rows16(uint32_t x) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return {r[0], r[1]};
}
__device__ __forceinline__ LanePair swap_rows32(uint32_t x) {
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return {r[0], r[1]};
}

// Value of lane ^ kMask, for the masks a butterfly or a mirror uses.
template <int kMask> __device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
    if constexpr (kMask == 0) return x;
    else if constexpr (kMask == 1) return dpp_move<0xB1>(x);   // quad_perm 1,0,3,2
    else if constexpr (kMask == 2) return dpp_move<0x4E>(x);   // quad_perm 2,3,0,1
    else if constexpr (kMask == 3) return dpp_move<0x1B>(x);   // quad_perm 3,2,1,0
    else if constexpr (kMask == 4) return dpp_move<0x141>(dpp_move<0x1B>(x));
    else if constexpr (kMask == 7) return dpp_move<0x141>(x);  // half-row mirror
    else if constexpr (kMask == 8) return dpp_move<0x128>(x);  // rotate a row by 8
    else if constexpr (kMask == 15) return dpp_move<0x140>(x); // row mirror
    else if constexpr (kMask == 16) {
        const LanePair p = swap_rows16(x);
        return (__lane_id() & 16) ? p.a : p.b;
    } else if constexpr (kMask == 32) {
        const LanePair p = swap_rows32(x);
        return (__lane_id() & 32) ? p.a : p.b;
    } else if constexpr (kMask == 31) return lane_xor<16>(lane_xor<15>(x));
    else {
        static_assert(kMask == 63, "unsupported lane mask");
        return lane_xor<32>(lane_xor<31>(x));
    }
}
template <int kMask> __device__ __forceinline__ uint64_t lane_xor64(uint64_t x) {
    return ((uint64_t)lane_xor<kMask>((uint32_t)(x >> 32)) << 32) | lane_xor<kMask>((uint32_t)x);
}

// Lane i's value, for an i that is the same in all lanes.
__device__ __forceinline__ uint64_t lane_u64(uint64_t x, uint32_t i) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), (int)i) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, (int)i);
}

// Minimum over each aligned group of G lanes, in every lane.
template <int G> __device__ __forceinline__ uint32_t group_min_u32(uint32_t x) {
    if constexpr (G >= 2) x = min(x, lane_xor<1>(x));
    if constexpr (G >= 4) x = min(x, lane_xor<2>(x));
    if constexpr (G >= 8) x = min(x, lane_xor<7>(x));    // quads hold one value each
    if constexpr (G >= 16) x = min(x, lane_xor<15>(x));  // so do half rows
    if constexpr (G >= 32) {
        const LanePair p = swap_rows16(x);
        x = min(p.a, p.b);
    }
    if constexpr (G >= 64) {
        const LanePair p = swap_rows32(x);
        x = min(p.a, p.b);
    }
    return x;
}
// 64-bit: the high halves first, then the low halves of their holders.
template <int G> __device__ __forceinline__ uint64_t group_min_u64(uint64_t x) {
    const uint32_t hi = (uint32_t)(x >> 32);
    const uint32_t mh = group_min_u32<G>(hi);
    const uint32_t ml = group_min_u32<G>(hi == mh ? (uint32_t)x : 0xFFFFFFFFu);
    return ((uint64_t)mh << 32) | ml;
}

// Inclusive prefix sum and prefix maximum over the wave's lanes (rows of 16 by
// shifts, then the row ends broadcast to the rows after them; lanes without a
// source add 0).
template <int kCtrl, int kRows> __device__ __forceinline__ uint32_t dpp_or_zero(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kCtrl, kRows, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_scan_sum(uint32_t x) {
    x += dpp_or_zero<0x111, 0xF>(x);  // row_shr 1, 2, 4, 8
    x += dpp_or_zero<0x112, 0xF>(x);
    x += dpp_or_zero<0x114, 0xF>(x);
    x += dpp_or_zero<0x118, 0xF>(x);
    x += dpp_or_zero<0x142, 0xA>(x);  // row_bcast 15 into rows 1 and 3
    x += dpp_or_zero<0x143, 0xC>(x);  // row_bcast 31 into rows 2 and 3
    return x;
}
__device__ __forceinline__ uint32_t wave_scan_max(uint32_t x) {
    x = max(x, dpp_or_zero<0x111, 0xF>(x));
    x = max(x, dpp_or_zero<0x112, 0xF>(x));
    x = max(x, dpp_or_zero<0x114, 0xF>(x));
    x = max(x, dpp_or_zero<0x118, 0xF>(x));
    x = max(x, dpp_or_zero<0x142, 0xA>(x));
    x = max(x, dpp_or_zero<0x143, 0xC>(x));
    return x;
}

// 64 x 64 bit transpose across the wave: bit j of lane i's result is bit i of
// lane j's argument.
template <int kStep> __device__ __forceinline__ uint64_t transpose_step(uint64_t x, uint64_t m) {
    const uint64_t y = lane_xor64<kStep>(x);
    return (__lane_id() & kStep) ? ((y >> kStep) & m) | (x & ~m) : (x & m) | ((y & m) << kStep);
}
__device__ __forceinline__ uint64_t wave_transpose(uint64_t x) {
    x = transpose_step<32>(x, 0x00000000FFFFFFFFull);
    x = transpose_step<16>(x, 0x0000FFFF0000FFFFull);
    x = transpose_step<8>(x, 0x00FF00FF00FF00FFull);
    x = transpose_step<4>(x, 0x0F0F0F0F0F0F0F0Full);
    x = transpose_step<2>(x, 0x3333333333333333ull);
    return transpose_step<1>(x, 0x5555555555555555ull);
}

// One compare-exchange step of a sorting network between lanes: the lane
// keeps the smaller (low) or the larger of its own value and its partner's.
__device__ __forceinline__ uint64_t keep_of(uint64_t own, uint64_t other, bool low) {
    return ((own < other) == low) ? own : other;
}

}  // namespace skim
