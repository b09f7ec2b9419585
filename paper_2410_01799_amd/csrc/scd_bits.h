// Lane exchanges on 32-bit words and the 64 x 64 bit transpose across a wave (shared by the kernels that contract
// over the terms of a decomposition, whose bitsets are term-major).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace scd {
namespace {

// (a, b) = the values of the two partners at distance D = 16 or 32, the same pair in both of them
template <int D>
__device__ __forceinline__ void swap_pair(uint32_t v, uint32_t& a, uint32_t& b)
{
    if constexpr (D == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        a = r[0], b = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        a = r[0], b = r[1];
    }
}
// 64 x 64 bit transpose across a wave: lane q brings row q (bit i = column i), lane i leaves with column i.
// Six butterfly stages (distance 32, 16, .., 1): in every 2s x 2s block the two off-diagonal s x s blocks
// change places, the partner row is s lanes away.  The rows are kept as two 32-bit halves; below distance
// 32 a stage is, per half, one lane exchange, one rotate (the partner's bits move s columns up in the
// upper row, s down in the lower) and one bitfield insert.  Distances 1..8 stay within a row of 16 lanes
// and use the data-parallel lane modes, distances 16 and 32 the row-swap instructions (no LDS traffic).
template <int S>
__device__ __forceinline__ uint32_t lane_xor_u32(uint32_t v, int lane)
{
    if constexpr (S == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);  // quad_perm 1,0,3,2
    else if constexpr (S == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);  // quad_perm 2,3,0,1
    else if constexpr (S == 4) {
        // lane ^ 7 (mirror of half a row), then lane ^ 3 (quad_perm 3,2,1,0)
        const int h = __builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true);
        return (uint32_t)__builtin_amdgcn_mov_dpp(h, 0x1B, 0xF, 0xF, true);
    } else if constexpr (S == 8) {
        // lane ^ 15 (mirror of a row), then lane ^ 7
        const int h = __builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, true);
        return (uint32_t)__builtin_amdgcn_mov_dpp(h, 0x141, 0xF, 0xF, true);
    } else {
        // distance 16 or 32: the row swap leaves (value of the lower partner, value of the upper partner) in
        // both lanes; each takes the other's
        uint32_t a, b;
        swap_pair<S>(v, a, b);
        return (lane & S) ? a : b;
    }
}

template <int S>
__device__ __forceinline__ uint32_t bit_butterfly(uint32_t h, int lane)
{
    constexpr uint32_t m = S == 16 ? 0x0000FFFFu : S == 8 ? 0x00FF00FFu : S == 4 ? 0x0F0F0F0Fu : S == 2 ? 0x33333333u : 0x55555555u;
    const bool lower = (lane & S) != 0;
    const uint32_t p = lane_xor_u32<S>(h, lane);
    const uint32_t rot = __builtin_amdgcn_alignbit(p, p, lower ? S : 32 - S);  // partner >> S (lower row), << S (upper)
    const uint32_t keep = lower ? ~m : m;
    return (h & keep) | (rot & ~keep);
}

__device__ __forceinline__ uint64_t transpose64(uint64_t x, int lane)
{
    uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
    {
        // distance 32: the upper rows take the partner's low half as their high half, the lower rows the
        // partner's high half as their low half
        const bool lower = (lane & 32) != 0;
        const uint32_t got = lane_xor_u32<32>(lower ? lo : hi, lane);
        lo = lower ? got : lo;
        hi = lower ? hi : got;
    }
    lo = bit_butterfly<16>(lo, lane), hi = bit_butterfly<16>(hi, lane);
    lo = bit_butterfly<8>(lo, lane), hi = bit_butterfly<8>(hi, lane);
    lo = bit_butterfly<4>(lo, lane), hi = bit_butterfly<4>(hi, lane);
    lo = bit_butterfly<2>(lo, lane), hi = bit_butterfly<2>(hi, lane);
    lo = bit_butterfly<1>(lo, lane), hi = bit_butterfly<1>(hi, lane);
    return ((uint64_t)hi << 32) | lo;
}

}  // namespace
}  // namespace scd
