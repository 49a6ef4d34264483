// bcf_cps.hip -- colored prefix sums on gfx950, the paper's example of how
// shared-memory bank conflicts decide a kernel's runtime (Sitchinava &
// Weichert, Sec. 1.2 and the appendix on colored prefix sums).
//
// out[i] = sum of values[j] over j <= i with colors[j] == colors[i] (inclusive,
// modulo 2^32), for d <= 32 colors, by the paper's three phases:
//   1. every work-group reduces its tile (a contiguous range, processed in
//      pages of 8192 elements) to d per-color sums;
//   2. one work-group per color scans those sums over the tiles: each tile's
//      starting offset per color;
//   3. every work-group scans its tile page by page: each thread counts the
//      32 consecutive elements it owns per color, the counts are scanned over
//      the threads per color (the intra-page offsets), and each thread then
//      walks its elements again with running per-color sums.
// The per-thread, per-color counters live in LDS (their color index is data,
// so they cannot be registers).  CF = false keeps a thread's d counters
// consecutive (word t * d + c): in one step the 32 lanes of a half-wave touch
// words t * d + c_t, whose banks collide more the larger d is -- the layout
// whose runtime grows with d in the paper.  CF = true stores them color-major
// (word c * 256 + t): lane t always hits bank t mod 32, whatever the colors,
// so every counter access is conflict-free, and the scans over threads run in
// registers (DPP row shifts and lane reads) instead of through a transposed
// LDS matrix.  The counters take 256 * d words of dynamic LDS, so small d
// leaves room for more resident work-groups.
//
// Both passes over the elements are bound by HBM, so what counts is how they
// read and write it: whole lines per instruction, in phase 3 through a
// transposition in LDS.  Measured at 2^26 elements and 16 colors: 250 us with
// every lane on its own 128 bytes, 203 so (one page per tile, 8192 tiles: 192, but
// the temp size is that of at most 2048 tiles).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bcf.h"

namespace {

constexpr int kThreads = 256;  // four waves per work-group
constexpr int kWaves = kThreads / 64;
constexpr int kPerThread = 32;  // consecutive elements a thread owns in a page
constexpr int kPage = kThreads * kPerThread;
constexpr uint32_t kMaxColors = 32;
constexpr uint64_t kMaxTiles = 2048;

template <bool CF>
__device__ __forceinline__ uint32_t slot(uint32_t t, uint32_t c, uint32_t d)
{
    return CF ? c * kThreads + t : t * d + c;
}

__device__ __forceinline__ uint32_t color_of(uint32_t c, uint32_t d) { return c < d ? c : d - 1; }

// Adds x to an LDS counter that no other thread touches: one instruction, and
// no wait for the old value.
__device__ __forceinline__ void counter_add(uint32_t *c, uint32_t x)
{
    __hip_atomic_fetch_add(c, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The values of a wave's 64 chunks of kPerThread consecutive elements, between
// global memory, where 8 lanes read or write a chunk's 128 bytes at once, and
// the registers of the lane that owns the chunk.  A lane on its own would touch
// 64 lines per instruction and come back to each eight times.  Half of every
// chunk passes through the wave's LDS at a time: chunk r's 16 words as four quads
// at words 16 r .. 16 r + 15, quad q at place q ^ ((r >> 1) & 3) ^ ((r >> 4) & 1).
// 16-byte writes go eight consecutive lanes at a time over 32 banks: there the
// first term spreads a lane per chunk's eight chunks.  16-byte reads go sixteen
// lanes at a time over 64 banks, in the groups {0-3, 12-15, 20-23, 24-27} and
// {4-11, 16-19, 28-31} of either half-wave: there the second term parts chunks 0-3
// from 24-27 and 4-7 from 28-31.  (Without it every second access of the load
// side's reads took two cycles more.)
typedef uint32_t Quad __attribute__((ext_vector_type(4)));
constexpr int kBatch = 4;                        // colors whose scans are in flight together
constexpr int kQuads = kPerThread / 4;           // 16-byte quads per chunk
constexpr uint32_t kStageWords = 64 * kPerThread / 2;  // per wave: 4 KiB

__device__ __forceinline__ Quad *stage_quad(uint32_t *stage, uint32_t row, uint32_t q)
{
    return reinterpret_cast<Quad *>(__builtin_assume_aligned(stage, 16)) + 4 * row + (q ^ ((row >> 1) & 3) ^ ((row >> 4) & 1));
}

__device__ __forceinline__ void load_values(const uint32_t *src, uint32_t *stage, uint32_t lane,
                                            uint32_t (&v)[kPerThread])
{
    const Quad *g = reinterpret_cast<const Quad *>(src);
    const uint32_t q = lane & 3, row = lane >> 2;  // of 16 rows per load
    Quad x[kQuads];
#pragma unroll
    for (int i = 0; i < kQuads; ++i)
        x[i] = g[kQuads * (16 * (i & 3) + row) + 4 * (i >> 2) + q];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *stage_quad(stage, 16 * i + row, q) = x[4 * h + i];
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const Quad y = *stage_quad(stage, lane, i);
            v[16 * h + 4 * i] = y.x;
            v[16 * h + 4 * i + 1] = y.y;
            v[16 * h + 4 * i + 2] = y.z;
            v[16 * h + 4 * i + 3] = y.w;
        }
        wave_lds_fence();
    }
}

__device__ __forceinline__ void store_values(uint32_t *dst, uint32_t *stage, uint32_t lane,
                                             const uint32_t (&v)[kPerThread])
{
    Quad *g = reinterpret_cast<Quad *>(dst);
    const uint32_t q = lane & 3, row = lane >> 2;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *stage_quad(stage, lane, i) =
                Quad{v[16 * h + 4 * i], v[16 * h + 4 * i + 1], v[16 * h + 4 * i + 2], v[16 * h + 4 * i + 3]};
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < 4; ++i)
            g[kQuads * (16 * i + row) + 4 * h + q] = *stage_quad(stage, 16 * i + row, q);
        wave_lds_fence();
    }
}

// The colors of the kPerThread elements a thread owns.
__device__ __forceinline__ void load_colors(const uint8_t *colors, uint32_t (&c)[kPerThread])
{
    const Quad *cp = reinterpret_cast<const Quad *>(colors);
#pragma unroll
    for (int q = 0; q < kPerThread / 16; ++q) {
        const Quad cc = cp[q];
        const uint32_t w[4] = {cc.x, cc.y, cc.z, cc.w};
#pragma unroll
        for (int i = 0; i < 16; ++i)
            c[16 * q + i] = (w[i / 4] >> (8 * (i % 4))) & 0xffu;
    }
}

// Inclusive prefix sum of x over the lanes of the wave, without LDS: a
// Kogge-Stone scan inside each row of 16 lanes by DPP row shifts (lanes with
// no source read 0), then each row adds the totals of the rows before it,
// read from lanes 15, 31 and 47.
__device__ __forceinline__ uint32_t wave_scan(uint32_t x, uint32_t lane)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);  // row_shr:8
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 15);
    const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 31);
    const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 47);
    const uint32_t row = lane >> 4;
    return x + (row > 0 ? r0 : 0u) + (row > 1 ? r1 : 0u) + (row > 2 ? r2 : 0u);
}

// Phase 1: per-color sums of tile b = [b * tile, min((b + 1) * tile, n)).
// The number of tiles is an argument here and below, not gridDim.x, which makes
// the host fill in the kernel's implicit arguments at every launch: calls of up
// to 10^6 elements are bound by the host's launches (21.4 us a call with gridDim.x, 20.8 so).
template <bool CF>
__global__ __launch_bounds__(kThreads) void k_cps_tile_sums(const uint32_t *values, const uint8_t *colors, uint64_t n,
                                                            uint32_t d, uint64_t tile, uint32_t tiles, uint32_t *sums)
{
    extern __shared__ uint32_t cnt[];  // kThreads * d counters
    __shared__ uint32_t part[kWaves][kMaxColors];
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t / 64;
    const uint64_t lo = (uint64_t)blockIdx.x * tile, hi = lo + tile < n ? lo + tile : n;
    for (uint32_t c = 0; c < d; ++c)
        cnt[slot<CF>(t, c, d)] = 0;
    // the order of the elements does not matter here: consecutive threads take
    // consecutive quads
    for (uint64_t page = lo; page < hi; page += kPage) {
        if (page + kPage <= hi) {
            const Quad *vp = reinterpret_cast<const Quad *>(values + page);
            const uint32_t *cp = reinterpret_cast<const uint32_t *>(colors + page);
            Quad x[kQuads];
            uint32_t cc[kQuads];
#pragma unroll
            for (int q = 0; q < kQuads; ++q) {
                x[q] = vp[kThreads * q + t];
                cc[q] = cp[kThreads * q + t];
            }
#pragma unroll
            for (int q = 0; q < kQuads; ++q) {
                const uint32_t v[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    counter_add(&cnt[slot<CF>(t, color_of((cc[q] >> (8 * i)) & 0xffu, d), d)], v[i]);
            }
        } else {
            for (uint64_t i = page + t; i < hi; i += kThreads)
                counter_add(&cnt[slot<CF>(t, color_of(colors[i], d), d)], values[i]);
        }
    }
    for (uint32_t c0 = 0; c0 < d; c0 += kBatch) {
        uint32_t x[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
            x[i] = cnt[slot<CF>(t, c0 + i < d ? c0 + i : c0, d)];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const uint32_t s = wave_scan(x[i], lane);
            if (lane == 63 && c0 + i < d)
                part[wave][c0 + i] = s;
        }
    }
    __syncthreads();
    if (t < d) {
        uint32_t s = 0;
        for (int w = 0; w < kWaves; ++w)
            s += part[w][t];
        sums[(uint64_t)t * tiles + blockIdx.x] = s;
    }
}

// Phase 2: work-group c turns the tile sums of color c into exclusive offsets
// (sums and offsets are color-major, so its loads are consecutive: 4.9 us for 2048
// tiles of 16 colors, 6.4 tile-major by 256 threads), with as many threads as the
// tiles need: 1.6 us for 7 tiles of one color, 1.8 with 1024 threads.
constexpr int kScanThreads = 1024;  // the most
constexpr int kScanPer = kMaxTiles / kScanThreads;  // consecutive tiles per thread, all loads in flight at once

__global__ __launch_bounds__(kScanThreads) void k_cps_tile_offsets(const uint32_t *sums, uint32_t *offsets,
                                                                   uint32_t tiles)
{
    __shared__ uint32_t wtot[kScanThreads / 64];
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t / 64, c = blockIdx.x;
    uint32_t x[kScanPer], local = 0;
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
        const uint32_t b = t * kScanPer + i;
        x[i] = b < tiles ? sums[(uint64_t)c * tiles + b] : 0;
    }
#pragma unroll
    for (int i = 0; i < kScanPer; ++i)
        local += x[i];
    const uint32_t incl = wave_scan(local, lane);
    if (lane == 63)
        wtot[wave] = incl;
    __syncthreads();
    uint32_t run = incl - local;
    for (uint32_t w = 0; w < wave; ++w)
        run += wtot[w];
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
        const uint32_t b = t * kScanPer + i;
        if (b < tiles)
            offsets[(uint64_t)c * tiles + b] = run;
        run += x[i];
    }
}

// Phase 3: the colored prefix sums of tile b, seeded with its offsets.
template <bool CF>
__global__ __launch_bounds__(kThreads) void k_cps_scan(const uint32_t *values, const uint8_t *colors, uint32_t *out,
                                                       uint64_t n, uint32_t d, uint64_t tile, uint32_t tiles,
                                                       const uint32_t *offsets)
{
    // from the last tile to the first: phase 1 left the end of the input in the
    // last-level cache (8 us of the call at 2^26 elements and 16 colors)
    const uint32_t bid = tiles - 1 - blockIdx.x;
    extern __shared__ uint32_t cnt[];  // kThreads * d counters
    __shared__ __align__(16) uint32_t stage_all[kWaves][kStageWords];
    __shared__ uint32_t wtot[kWaves][kMaxColors];
    __shared__ uint32_t carry[kMaxColors];
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t / 64;
    const uint64_t lo = (uint64_t)bid * tile, hi = lo + tile < n ? lo + tile : n;
    if (t < d)
        carry[t] = offsets[(uint64_t)t * tiles + bid];
    for (uint64_t page = lo; page < hi; page += kPage) {
        const uint64_t base = page + (uint64_t)t * kPerThread;
        const uint64_t wbase = page + (uint64_t)wave * (64 * kPerThread);
        const bool whole = wbase + 64 * kPerThread <= hi;  // the wave's chunks, all in range
        const uint32_t valid = whole || base + kPerThread <= hi ? kPerThread : base < hi ? (uint32_t)(hi - base) : 0u;
        uint32_t v[kPerThread], col[kPerThread];
        if (whole) {
            load_colors(colors + base, col);
            load_values(values + wbase, stage_all[wave], lane, v);
        } else {
#pragma unroll
            for (int i = 0; i < kPerThread; ++i) {
                const bool in = (uint32_t)i < valid;
                v[i] = in ? values[base + i] : 0u;
                col[i] = in ? colors[base + i] : 0u;
            }
        }
#pragma unroll
        for (int i = 0; i < kPerThread; ++i)
            col[i] = color_of(col[i], d);
        // this thread's per-color sums of its kPerThread elements
        for (uint32_t c = 0; c < d; ++c)
            cnt[slot<CF>(t, c, d)] = 0;
#pragma unroll
        for (int i = 0; i < kPerThread; ++i)
            counter_add(&cnt[slot<CF>(t, col[i], d)], v[i]);  // past the end: 0
        // exclusive scan over the threads, per color: within the wave in
        // registers, then across the four waves
        for (uint32_t c0 = 0; c0 < d; c0 += kBatch) {
            uint32_t x[kBatch];
#pragma unroll
            for (int i = 0; i < kBatch; ++i)
                x[i] = cnt[slot<CF>(t, c0 + i < d ? c0 + i : c0, d)];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                const uint32_t incl = wave_scan(x[i], lane);
                if (c0 + i < d) {
                    cnt[slot<CF>(t, c0 + i, d)] = incl - x[i];
                    if (lane == 63)
                        wtot[wave][c0 + i] = incl;
                }
            }
        }
        __syncthreads();
        for (uint32_t c = 0; c < d; ++c) {
            uint32_t base = carry[c];
            for (uint32_t w = 0; w < wave; ++w)
                base += wtot[w][c];
            counter_add(&cnt[slot<CF>(t, c, d)], base);
        }
        __syncthreads();
        if (t < d) {
            uint32_t s = 0;
            for (int w = 0; w < kWaves; ++w)
                s += wtot[w][t];
            carry[t] += s;
        }
        // running sums over this thread's elements
        uint32_t r[kPerThread];
#pragma unroll
        for (int i = 0; i < kPerThread; ++i)  // past the end: 0 is added
            r[i] = v[i] + __hip_atomic_fetch_add(&cnt[slot<CF>(t, col[i], d)], v[i], __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
        if (whole) {
            store_values(out + wbase, stage_all[wave], lane, r);
        } else {
#pragma unroll
            for (int i = 0; i < kPerThread; ++i)
                if ((uint32_t)i < valid)
                    out[base + i] = r[i];
        }
        __syncthreads();  // the next page reuses the counters and wtot
    }
}

// Tiles of a call over n > 0 elements: at most kMaxTiles, each a multiple of a
// page (kPage elements).
void tiling(uint64_t n, uint64_t &tiles, uint64_t &tile)
{
    const uint64_t pages = (n + kPage - 1) / kPage;
    const uint64_t per = (pages + kMaxTiles - 1) / kMaxTiles;  // pages per tile
    tile = per * kPage;
    tiles = (n + tile - 1) / tile;
}

}  // namespace

extern "C" bcf_status bcf_colored_prefix_sums(const uint32_t *values, const uint8_t *colors, uint32_t *out,
                                              uint64_t n, uint32_t d, int conflict_free, void *temp,
                                              uint64_t *temp_bytes, void *stream)
{
    if (!temp_bytes || d == 0 || d > kMaxColors || n > 0xffffffffull)
        return BCF_ERR_INVALID;
    if (n == 0) {
        if (!temp)
            *temp_bytes = 0;
        return BCF_OK;
    }
    uint64_t tiles = 0, tile = 0;
    tiling(n, tiles, tile);
    const uint64_t sums_bytes = (tiles * d * 4 + 255) / 256 * 256;
    const uint64_t need = 2 * sums_bytes;
    if (!temp) {
        *temp_bytes = need;
        return BCF_OK;
    }
    if (!values || !colors || !out)
        return BCF_ERR_INVALID;
    if (((reinterpret_cast<uintptr_t>(values) | reinterpret_cast<uintptr_t>(colors) |
          reinterpret_cast<uintptr_t>(out)) & 15) != 0)
        return BCF_ERR_INVALID;  // 16-byte accesses
    if (*temp_bytes < need)
        return BCF_ERR_TEMP_TOO_SMALL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint32_t *sums = static_cast<uint32_t *>(temp);
    uint32_t *offsets = reinterpret_cast<uint32_t *>(static_cast<char *>(temp) + sums_bytes);
    const dim3 grid((uint32_t)tiles), block(kThreads);
    const size_t lds = (size_t)kThreads * d * sizeof(uint32_t);
    if (conflict_free)
        hipLaunchKernelGGL(k_cps_tile_sums<true>, grid, block, lds, s, values, colors, n, d, tile, (uint32_t)tiles,
                           sums);
    else
        hipLaunchKernelGGL(k_cps_tile_sums<false>, grid, block, lds, s, values, colors, n, d, tile, (uint32_t)tiles,
                           sums);
    const uint32_t scan_threads = (uint32_t)((tiles + 64 * kScanPer - 1) / (64 * kScanPer) * 64);
    hipLaunchKernelGGL(k_cps_tile_offsets, dim3(d), dim3(scan_threads), 0, s, sums, offsets, (uint32_t)tiles);
    if (conflict_free)
        hipLaunchKernelGGL(k_cps_scan<true>, grid, block, lds, s, values, colors, out, n, d, tile,
                           (uint32_t)tiles, offsets);
    else
        hipLaunchKernelGGL(k_cps_scan<false>, grid, block, lds, s, values, colors, out, n, d, tile,
                           (uint32_t)tiles, offsets);
    return hipGetLastError() == hipSuccess ? BCF_OK : BCF_ERR_DEVICE;
}
