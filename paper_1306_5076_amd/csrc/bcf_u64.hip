// bcf_u64.hip -- sort of unsigned 64-bit keys (an extension: the paper sorts
// 32-bit keys) on the same design as the 32-bit sort, with a key held in a
// register pair and compared as one 64-bit integer.
//
// * Block sort (the paper's base case, Sec. 3.1): up to 6 M keys, four waves sort a
//   tile of 4096 keys with 16 keys per lane (the networks of the small 32-bit
//   sorts).  Above, four waves sort 16384 keys: each lane sorts a line of 64
//   with Batcher's odd-even merge sort, six merge rounds turn a wave's 64 lines
//   into one run of 4096 keys, and two more rounds through the shared CROSS
//   layout merge the waves' runs.  Layout changes go through LDS as two 32-bit
//   halves, each with the conflict-free rows of the 32-bit tiles.
// * Merge passes (Sec. 3.2, binary merging): every work-group produces 8192
//   outputs of one merge of two runs, every wave 2048 of them.  Co-ranks (the
//   merge-path split, exact whatever the duplicates) bound each tile's pieces,
//   the A piece is loaded ascending and the B piece reversed into one bitonic
//   tile, a half-cleaner network sorts it and the tile is stored coalesced.
//   Passes ping-pong between the output and temp so that the last one writes
//   the output.
// Keys only: equal keys are indistinguishable, so the order among them needs
// no tie-break.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bcf.h"
#include "bcf_device.hpp"
#include "bcf_tile16.hpp"

namespace bcf {

// Host services of bcf_api.hip: a profiling scope around one launch.
void *prof_begin(const char *name, hipStream_t s, double bytes);
void prof_end(void *scope);

namespace {

constexpr uint64_t kMaxN64 = 0xFFFFFFFFull;

// STRIDED tile of `count` keys from src (position p = 64 r + lane), padding
// with the maximum key (never stored).
__device__ __forceinline__ void load_tile64(Lines64 &t, const uint64_t *__restrict__ src, uint32_t count,
                                            uint32_t lane)
{
    if (count >= (uint32_t)kTile) {
#pragma unroll
        for (int r = 0; r < kLine; ++r)
            t.e[r] = src[kWave * r + lane];
        return;
    }
    const uint32_t last = count ? count - 1 : 0;
#pragma unroll
    for (int r = 0; r < kLine; ++r) {
        const uint32_t p = kWave * r + lane;
        const uint64_t k = count ? src[p < count ? p : last] : kMaxKey64;  // clamped: a valid address
        t.e[r] = p < count ? k : kMaxKey64;
    }
}

// Loads and stores of a pass, with the nontemporal hint when the pass
// streams more than the last-level cache holds (below that the next pass
// finds its input there).
template <bool NT>
__device__ __forceinline__ uint64_t ld64(const uint64_t *p)
{
    if constexpr (NT)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

template <bool NT>
__device__ __forceinline__ void store_tile64(const Lines64 &t, uint64_t *__restrict__ dst, uint32_t count,
                                             uint32_t lane)
{
#pragma unroll
    for (int r = 0; r < kLine; ++r) {
        const uint32_t p = kWave * r + lane;
        if (p < count) {
            if constexpr (NT)
                __builtin_nontemporal_store(t.e[r], dst + p);
            else
                dst[p] = t.e[r];
        }
    }
}

constexpr int kGroupWaves64 = 4;  // group tiles of 16384 keys
// Sorts of more keys than this take group tiles.  Four-wave tiles and two more
// merge passes against group tiles: 2^20 keys 144 / 206 us, 2^22 230 / 257, 6 M 318 /
// 337, 2^23 405 / 397.
constexpr uint64_t kGroupMinN64 = 6ull << 20;

// One 4096-key tile per work-group of four waves, 16 keys per lane, for sorts of at
// most kGroupMinN64 keys: a wave with 64 keys per lane takes 53 us for its chain of
// instructions, which nothing hides where the chip is nearly empty.
__global__ __launch_bounds__(kSmallThreads) void k_u64_tile_sort(const uint64_t *__restrict__ in,
                                                                 uint64_t *__restrict__ out, uint64_t n)
{
    constexpr int N = kSmallLine;
    __shared__ __align__(16) uint32_t lds[2][2 * kTile];
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint64_t start = (uint64_t)blockIdx.x * kTile;
    if (start >= n)
        return;
    const uint32_t count = n - start < (uint64_t)kTile ? (uint32_t)(n - start) : (uint32_t)kTile;
    Lines64 t{};
#pragma unroll
    for (int r = 0; r < N; ++r) {
        const uint32_t p = kSmallThreads * r + tid;
        const uint64_t k = in[start + (p < count ? p : count - 1)];  // clamped: a valid address
        t.e[r] = p < count ? k : kMaxKey64;
    }
    small_sort(t, lds[0], lds[1], wave, lane);
    // through LDS, so that consecutive lanes store consecutive keys: position p at
    // word pair p ^ (p / 16 mod 16), which spreads a lane's 16 keys over the banks
    uint64_t *stage = reinterpret_cast<uint64_t *>(lds[1]);
#pragma unroll
    for (int r = 0; r < N; ++r)
        stage[N * tid + (r ^ (tid & (N - 1)))] = t.e[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < N; ++r) {
        const uint32_t p = kSmallThreads * r + tid;
        if (p < count)
            out[start + p] = stage[p ^ ((p / N) & (N - 1))];
    }
}

// One group tile of kGroupWaves64 sub-tiles per work-group: each wave sorts
// its sub-tile (odd waves descending, by complementing around the sort), then
// the group rounds merge across the waves.  Every wave of a work-group reaches
// the same barriers: waves whose sub-tile lies past the end hold padding only.
// Two waves per SIMD; 24 registers spill (64 bytes of scratch per lane).
template <bool NT>
__global__ __launch_bounds__(kWave *kGroupWaves64) __attribute__((amdgpu_waves_per_eu(2))) void k_u64_block_sort_group(
    const uint64_t *__restrict__ in, uint64_t *__restrict__ out, uint64_t n)
{
    __shared__ __align__(16) uint32_t lds[kGroupWaves64 * kLdsWords];
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint64_t gstart = (uint64_t)blockIdx.x * (kGroupWaves64 * kTile);
    if (gstart >= n)
        return;
    const uint64_t start = gstart + (uint64_t)wave * kTile;
    const uint32_t count = start >= n ? 0u : (n - start < (uint64_t)kTile ? (uint32_t)(n - start) : (uint32_t)kTile);
    Lines64 t;
    load_tile64(t, in + start, count, lane);  // count 0: padding only, nothing loaded
    uint32_t *own = lds + kLdsWords * wave;
    if (count != 0) {  // else padding only
        flip(t, wave);
        sort_tile_wide(t, own, lane);
        flip(t, wave);
    }
    group_rounds<kGroupWaves64, 7>(t, lds, lane, wave);
    to_strided(t, own, lane);
    store_tile64<NT>(t, out + start, count, lane);
}

// A merge tile holds 2048 keys, 32 per lane: the registers of four waves per
// SIMD.  Four waves of a work-group take four consecutive tiles: one search over
// the runs per 8192 keys, the inner ones inside the work-group's own pieces.  A
// pass is bound by its chain of loads and by the lines its searches fetch: a
// search of its own per tile fetched as much as the keys.  Measured at 12,000,001
// keys, per pass under the profiler: 57 us with 4096 keys per wave or with 2048,
// 44 so (4.3 TB/s); the sort 776 -> 634 us.
constexpr int kMergeLine = 32;
constexpr int kMergeKeys = kMergeLine * kWave;
constexpr int kMergeWaves = 4;                   // tiles of a work-group
constexpr int kMergeStride = 36;  // LDS words per 32 positions: 16-byte rows of 8 lanes cover the 32 banks
constexpr int kMergeLdsWords = kMergeKeys / 32 * kMergeStride;

__device__ __forceinline__ void cx64(uint64_t &a, uint64_t &b)
{
    const uint64_t x = a, y = b;
    const bool lt = x < y;
    a = lt ? x : y;
    b = lt ? y : x;
}

// Half-cleaner steps at register distances D, D/2, ..., 1.
template <int D>
__device__ __forceinline__ void clean32(uint64_t (&x)[kMergeLine])
{
#pragma unroll
    for (int r = 0; r < kMergeLine; ++r)
        if ((r & D) == 0)
            cx64(x[r], x[r + D]);
    if constexpr (D > 1)
        clean32<D / 2>(x);
}

// The word of both halves that `at` (0: low, 32: high) names.
__device__ __forceinline__ uint32_t word_of(uint64_t x, int at) { return (uint32_t)(x >> at); }

// Sorts a bitonic tile: on entry and exit position 64 r + lane in register r.
// Position bits 10..6 are register bits; bit 5 (lane bit 5) meets through an
// exchange of the half-waves of two registers, after which lane bit 5 holds
// position bit 10 and register bit 4 position bit 5; bits 4..0 are register
// bits once position 32 lane + r is in register r.
__device__ __forceinline__ void merge_tile64(uint64_t (&x)[kMergeLine], uint32_t *lds, uint32_t lane)
{
    constexpr int H = kMergeLine / 2;
    clean32<H>(x);
#pragma unroll
    for (int r = 0; r < H; ++r) {
        const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x[r], (uint32_t)x[r + H], false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x[r] >> 32), (uint32_t)(x[r + H] >> 32), false, false);
        x[r] = ((uint64_t)hi[0] << 32) | lo[0];
        x[r + H] = ((uint64_t)hi[1] << 32) | lo[1];
        cx64(x[r], x[r + H]);
    }
    uint32_t *half = lds + kMergeStride * (32 * (lane >> 5)) + (lane & 31);    // rows of p bit 10
    uint32_t *pairs = lds + kMergeStride * (lane >> 5) + (lane & 31);          // rows of p bit 5
    uint32_t *row = static_cast<uint32_t *>(__builtin_assume_aligned(lds + kMergeStride * lane, 16));
    uint32_t w[2][kMergeLine];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int r = 0; r < kMergeLine; ++r)
            half[kMergeStride * (2 * (r % H) + r / H)] = word_of(x[r], 32 * h);
        wave_lds_fence();
#pragma unroll
        for (int r = 0; r < kMergeLine; ++r)
            w[h][r] = row[r];
        wave_lds_fence();
    }
#pragma unroll
    for (int r = 0; r < kMergeLine; ++r)
        x[r] = ((uint64_t)w[1][r] << 32) | w[0][r];
    clean32<H>(x);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int r = 0; r < kMergeLine; ++r)
            row[r] = word_of(x[r], 32 * h);
        wave_lds_fence();
#pragma unroll
        for (int r = 0; r < kMergeLine; ++r)
            w[h][r] = pairs[2 * kMergeStride * r];
        wave_lds_fence();
    }
#pragma unroll
    for (int r = 0; r < kMergeLine; ++r)
        x[r] = ((uint64_t)w[1][r] << 32) | w[0][r];
}

// Output tile t of a binary pass over runs of `run` keys (a multiple of
// 4096): runs 2s and 2s+1 merge into [2s run, min(2(s+1) run, n)).
template <bool NT>
__global__ __launch_bounds__(kWave *kMergeWaves) __attribute__((amdgpu_waves_per_eu(4))) void k_u64_merge(
    const uint64_t *__restrict__ src, uint64_t *__restrict__ dst, uint64_t n, uint64_t run)
{
    __shared__ __align__(16) uint32_t lds_all[kMergeWaves][kMergeLdsWords];
    __shared__ uint32_t cut[kMergeWaves + 1];
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t *lds = lds_all[wave];
    uint64_t gstart = (uint64_t)blockIdx.x * (kMergeWaves * kMergeKeys);
    if (gstart >= n)
        return;
    const uint64_t base = gstart / (2 * run) * (2 * run);
    const uint64_t rem = n - base;
    const uint32_t na = (uint32_t)(rem < run ? rem : run);
    const uint32_t nb = (uint32_t)(rem - na < run ? rem - na : run);
    const uint32_t g0 = (uint32_t)(gstart - base);
    const uint32_t gcount = min(na + nb - g0, (uint32_t)(kMergeWaves * kMergeKeys));
    const uint64_t *A = src + base, *B = A + na;
    // the work-group's co-ranks (lanes 0..31: of its first output, 32..63: of its
    // end), then those of its inner tiles, inside the pieces it is going to load
    if (wave == 0) {
        const uint32_t split = corank_halfwave(A, na, B, nb, lane < 32 ? g0 : g0 + gcount, lane);
        if ((lane & 31) == 0)
            cut[lane < 32 ? 0 : kMergeWaves] = split;
    }
    __syncthreads();
    if (wave != 0) {
        const uint32_t ga = cut[0], gpa = cut[kMergeWaves] - ga;
        const uint32_t d = min(wave * kMergeKeys, gcount);
        const uint32_t split = corank_halfwave(A + ga, gpa, B + (g0 - ga), gcount - gpa, d, lane);
        if (lane == 0)
            cut[wave] = ga + split;
    }
    __syncthreads();
    if (wave * kMergeKeys >= gcount)
        return;
    const uint32_t a0 = uniform(cut[wave]), a1 = uniform(cut[wave + 1]);
    const uint32_t d0 = g0 + wave * kMergeKeys, count = min(gcount - wave * kMergeKeys, (uint32_t)kMergeKeys);
    gstart += wave * kMergeKeys;
    const uint32_t pa = a1 - a0, pb = count - pa;
    // A piece ascending at [0, pa), B piece reversed at [2048 - pb, 2048):
    // position p reads pA[p] or pA[bend - p], the B piece lying dB keys after
    // the A piece; one 32-bit offset per register, every load issued before
    // any is used
    const uint64_t *pA = A + a0;
    const uint32_t dB = na - a0 + (d0 - a0);
    const uint32_t bend = dB + (kMergeKeys - 1);
    const uint32_t bstart = kMergeKeys - pb;
    uint64_t x[kMergeLine];
    if (count == (uint32_t)kMergeKeys) {
        // full tile: every position is in A or in B, no select after a load
#pragma unroll
        for (int r = 0; r < kMergeLine; ++r) {
            const uint32_t p = kWave * r + lane;
            x[r] = ld64<NT>(pA + (p < pa ? p : bend - p));
        }
    } else {
#pragma unroll
        for (int r = 0; r < kMergeLine; ++r) {
            const uint32_t p = kWave * r + lane;
            const bool in_a = p < pa, in_b = p >= bstart;
            const uint64_t k = ld64<NT>(pA + (in_a ? p : (in_b ? bend - p : 0u)));
            x[r] = (in_a || in_b) ? k : kMaxKey64;
        }
    }
    merge_tile64(x, lds, lane);
    uint64_t *out = dst + gstart;
#pragma unroll
    for (int r = 0; r < kMergeLine; ++r) {
        const uint32_t p = kWave * r + lane;
        if (p < count) {
            if constexpr (NT)
                __builtin_nontemporal_store(x[r], out + p);
            else
                out[p] = x[r];
        }
    }
}

uint64_t align256(uint64_t b) { return (b + 255) / 256 * 256; }

// Run length after the block sort, and the binary merge passes after it.
uint64_t run0_for(uint64_t n) { return n > kGroupMinN64 ? (uint64_t)kGroupWaves64 * kTile : (uint64_t)kTile; }

uint32_t passes_for(uint64_t n)
{
    uint32_t p = 0;
    const uint64_t run0 = run0_for(n);
    for (uint64_t runs = (n + run0 - 1) / run0; runs > 1; runs = (runs + 1) / 2)
        ++p;
    return p;
}

}  // namespace
}  // namespace bcf

using namespace bcf;

extern "C" bcf_status bcf_sort_u64(const uint64_t *keys_in, uint64_t *keys_out, uint64_t n, void *temp,
                                   uint64_t *temp_bytes, void *stream)
{
    if (!temp_bytes || n > kMaxN64)
        return BCF_ERR_INVALID;
    const uint32_t passes = passes_for(n);
    const uint64_t need = passes ? align256(n * sizeof(uint64_t)) : 0;  // the ping-pong buffer
    if (!temp) {
        *temp_bytes = need;
        return BCF_OK;
    }
    if (n == 0)
        return BCF_OK;
    if (!keys_in || !keys_out)
        return BCF_ERR_INVALID;
    if (*temp_bytes < need)
        return BCF_ERR_TEMP_TOO_SMALL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint64_t *tb = static_cast<uint64_t *>(temp);
    // buffer after pass j: the output when passes - j is even, so the last pass writes it
    auto buf = [&](uint32_t j) { return ((passes - j) % 2 == 0) ? keys_out : tb; };
    const uint32_t tiles = (uint32_t)((n + kTile - 1) / kTile);
    // MI355X's last-level cache holds 256 MiB; a pass reads and writes 16 B per key
    const bool nt = 16.0 * n > 256.0 * 1024 * 1024;
    const uint64_t run0 = run0_for(n);
    void *scope = prof_begin("block_sort_u64", s, 16.0 * n);
    if (run0 > (uint64_t)kTile) {
        const uint32_t groups = (uint32_t)((n + run0 - 1) / run0);
        const dim3 block(kWave * kGroupWaves64);
        if (nt)
            hipLaunchKernelGGL(k_u64_block_sort_group<true>, dim3(groups), block, 0, s, keys_in, buf(0), n);
        else
            hipLaunchKernelGGL(k_u64_block_sort_group<false>, dim3(groups), block, 0, s, keys_in, buf(0), n);
    } else {
        hipLaunchKernelGGL(k_u64_tile_sort, dim3(tiles), dim3(kSmallThreads), 0, s, keys_in, buf(0), n);
    }
    prof_end(scope);
    if (hipGetLastError() != hipSuccess)
        return BCF_ERR_DEVICE;
    constexpr uint32_t kMergeGroup = kMergeWaves * kMergeKeys;
    const uint32_t merge_groups = (uint32_t)((n + kMergeGroup - 1) / kMergeGroup);
    uint64_t run = run0;
    for (uint32_t j = 1; j <= passes; ++j, run *= 2) {
        scope = prof_begin("merge_u64", s, 16.0 * n);
        if (nt)
            hipLaunchKernelGGL(k_u64_merge<true>, dim3(merge_groups), dim3(kWave * kMergeWaves), 0, s, buf(j - 1), buf(j), n, run);
        else
            hipLaunchKernelGGL(k_u64_merge<false>, dim3(merge_groups), dim3(kWave * kMergeWaves), 0, s, buf(j - 1), buf(j), n, run);
        prof_end(scope);
        if (hipGetLastError() != hipSuccess)
            return BCF_ERR_DEVICE;
    }
    return BCF_OK;
}
