// Networks of a 4096-element tile held by four waves, 16 elements per lane, for
// tiles whose time is one wave's chain of instructions: a quarter of the chain of
// the 64-element lines, without transposes.
#pragma once

#include <type_traits>

#include "bcf_device.hpp"

namespace bcf {

constexpr int kSmallWaves = 4;
constexpr int kSmallThreads = kSmallWaves * kWave;
constexpr int kSmallLine = kTile / kSmallThreads;  // 16 elements per lane
static_assert(kSmallLine == 16, "the register networks below");

// x of lane (lane ^ MASK), MASK below 64.  Within a row of 16 lanes by DPP
// moves, within 32 lanes by the LDS crossbar (ds_swizzle, no LDS memory), else
// by ds_bpermute.
template <int MASK>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x, uint32_t lane)
{
    if constexpr (MASK == 1)
        return dpp_move<kDppXor1>(x);
    else if constexpr (MASK == 2)
        return dpp_move<kDppXor2>(x);
    else if constexpr (MASK == 3)
        return dpp_move<kDppXor3>(x);
    else if constexpr (MASK == 4)
        return dpp_move<kDppXor3>(dpp_move<kDppXor7>(x));
    else if constexpr (MASK == 7)
        return dpp_move<kDppXor7>(x);
    else if constexpr (MASK == 8)
        return dpp_move<0x128>(x);  // row_ror:8
    else if constexpr (MASK == 15)
        return dpp_move<0x140>(x);  // row_mirror
    else if constexpr (MASK < 32)
        return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, (MASK << 10) | 0x1f);
    else
        return (uint32_t)__builtin_amdgcn_ds_bpermute((int)((lane ^ MASK) * 4), (int)x);
}
template <int MASK>
__device__ __forceinline__ uint64_t lane_xor(uint64_t x, uint32_t lane)
{
    const uint32_t hi = lane_xor<MASK>((uint32_t)(x >> 32), lane), lo = lane_xor<MASK>((uint32_t)x, lane);
    return ((uint64_t)hi << 32) | lo;
}
template <int MASK>
__device__ __forceinline__ double lane_xor(double x, uint32_t lane)
{
    return elem_of(lane_xor<MASK>(bits_of(x), lane));
}

// The smaller of x and y where `keep` is 0, the larger where it is ~0.
__device__ __forceinline__ uint32_t keep_one(uint32_t x, uint32_t y, uint32_t keep) { return med3(x, y, keep); }
template <class E>
__device__ __forceinline__ E keep_one(E x, E y, uint32_t keep)
{
    return ((x < y) != (keep != 0)) ? x : y;  // equal elements are alike in every bit
}

__device__ __forceinline__ uint32_t word_bits(uint32_t x) { return x; }
__device__ __forceinline__ uint64_t word_bits(uint64_t x) { return x; }
__device__ __forceinline__ uint64_t word_bits(double x) { return bits_of(x); }
__device__ __forceinline__ void from_bits(uint32_t &x, uint32_t b) { x = b; }
__device__ __forceinline__ void from_bits(uint64_t &x, uint64_t b) { x = b; }
__device__ __forceinline__ void from_bits(double &x, uint64_t b) { x = elem_of(b); }

// One stage against lane ^ MASK; with MIRROR against its mirrored register.
template <int MASK, bool MIRROR, class L>
__device__ __forceinline__ void small_lane_clean(L &t, uint32_t lane)
{
    constexpr int kTop = MASK & ~(MASK >> 1);  // highest bit: its holders keep the larger
    const uint32_t keep = opaque((lane & kTop) ? ~0u : 0u);
    auto &x = elems(t);
    typename std::remove_reference<decltype(x[0])>::type y[kSmallLine];
#pragma unroll
    for (int r = 0; r < kSmallLine; ++r)
        y[r] = lane_xor<MASK>(x[MIRROR ? kSmallLine - 1 - r : r], lane);
#pragma unroll
    for (int r = 0; r < kSmallLine; ++r)
        x[r] = keep_one(x[r], y[r], keep);
}

// The stages on lane bits B .. 0 and on the registers that end every round.
template <int B, class L>
__device__ __forceinline__ void small_lanes_down(L &t, uint32_t lane)
{
    if constexpr (B >= 0) {
        small_lane_clean<(1 << (B < 0 ? 0 : B)), false>(t, lane);
        small_lanes_down<B - 1>(t, lane);
    } else {
        half_clean_lines<kSmallLine / 2, -1>(t);
    }
}

// Round J (1..6): lanes l and l ^ (2^J - 1) hold mirrored places of two
// ascending runs.
template <int J, class L>
__device__ __forceinline__ void small_round(L &t, uint32_t lane)
{
    small_lane_clean<(1 << J) - 1, true>(t, lane);
    small_lanes_down<J - 2>(t, lane);
}

// The same stage against wave ^ mask, through LDS words [wave][register][lane].
template <bool MIRROR, class L>
__device__ __forceinline__ void small_wave_clean(L &t, uint32_t *buf, uint32_t wave, uint32_t mask, uint32_t lane)
{
    constexpr int N = kSmallLine;
    const uint32_t other = wave ^ mask;
    const uint32_t keep = wave > other ? ~0u : 0u;
    uint32_t *w = buf + wave * N * kWave + lane;
    const uint32_t *rd = buf + other * N * kWave + (MIRROR ? kWave - 1 - lane : lane);
    auto &x = elems(t);
    using E = typename std::remove_reference<decltype(x[0])>::type;
    constexpr bool kWide = sizeof(E) == 8;  // both halves, one after the other in the buffer
#pragma unroll
    for (int r = 0; r < N; ++r) {
        const auto b = word_bits(x[r]);
        w[r * kWave] = (uint32_t)b;
        if constexpr (kWide)
            w[kTile + r * kWave] = (uint32_t)(b >> 32);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < N; ++r) {
        const int q = (MIRROR ? N - 1 - r : r) * kWave;
        E y;
        if constexpr (kWide)
            from_bits(y, ((uint64_t)rd[kTile + q] << 32) | rd[q]);
        else
            from_bits(y, rd[q]);
        x[r] = keep_one(x[r], y, keep);
    }
}

// Sorts a tile: on entry any order, on exit position 16 (64 wave + lane) + r in
// register r.  lds0 and lds1 hold the tile's words (twice as many for 64-bit
// elements); lds1 is written after the first barrier and free after the last.
template <class L>
__device__ __forceinline__ void small_sort(L &t, uint32_t *lds0, uint32_t *lds1, uint32_t wave, uint32_t lane)
{
    oe_sort_lines<0, kSmallLine - 1>(t);
    small_round<1>(t, lane);
    small_round<2>(t, lane);
    small_round<3>(t, lane);
    small_round<4>(t, lane);
    small_round<5>(t, lane);
    small_round<6>(t, lane);
    small_wave_clean<true>(t, lds0, wave, 1, lane);
    small_lanes_down<5>(t, lane);
    small_wave_clean<true>(t, lds1, wave, 3, lane);
    // the first buffer again: every wave has read it before the barrier above
    small_wave_clean<false>(t, lds0, wave, 1, lane);
    small_lanes_down<5>(t, lane);
}

}  // namespace bcf
