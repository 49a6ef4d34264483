// Device code of small sorts (a few hundred 4096-element tiles at most), where
// the chip is nearly empty and the time is the latency of one wave's chain of
// instructions and of the launches after it:
//   k_tile_sort   -- the block sort of a tile by four waves with 16 elements per
//                    lane, a quarter of the chain of the 64-element lines;
//   k_rank_merge  -- a merge pass of up to 16 runs at once: every element's place
//                    is its own index plus its ranks in the other runs.
// Included by bcf_kernels.hip (it uses the key maps and samples defined there).
#pragma once

#include "bcf_tile16.hpp"

namespace bcf {

typedef uint32_t Quad __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes at any word

// One 4096-element tile per work-group of four waves, 16 elements per lane.
// Position bits: 0..3 registers, 4..9 lanes, 10..11 waves.  Ascending mirrored
// rounds as in sort_tile_keys; every stage between lanes takes about two VALU
// instructions per key (five per key/value element), so in all a tile costs
// half as many instructions again as the 64-element lines, but a wave's chain
// is a quarter as long, without transposes.  Measured for one tile:
// 13.1 us as one wave of 64-element lines, 6.6 us so (key/value: 33 and 17 us).
template <bool P, class Src>
__global__ __launch_bounds__(kSmallThreads) void k_tile_sort(Src src)
{
    constexpr int N = kSmallLine;
    __shared__ __align__(16) uint32_t lds[2][(P ? 2 : 1) * kTile];
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const SortItem it = src.get(blockIdx.x);
    const uint32_t count = uniform(it.count);
    const uint32_t pad = pad_key(src);
    Lines<P> t{};
    uint32_t vals[N];
    {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(uniform(it.ks)),
                                                                            (short)0, (int)(count * 4u), 0x00020000);
        uint32_t key[N];
#pragma unroll
        for (int r = 0; r < N; ++r)
            key[r] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(4u * (kSmallThreads * r + tid)), 0, 0);
        if constexpr (P) {
            const __amdgpu_buffer_rsrc_t vs = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<uint32_t *>(uniform(it.vs)), (short)0, (int)(count * 4u), 0x00020000);
#pragma unroll
            for (int r = 0; r < N; ++r)
                vals[r] =
                    (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(vs, (int)(4u * (kSmallThreads * r + tid)), 0, 0);
        }
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const uint32_t p = kSmallThreads * r + tid;
            uint32_t k = p < count ? key[r] : pad;
            if constexpr (Src::kMapped)
                k = map_key(k, src.in_map.sign, src.in_map.rest, src.in_map.inverse);
            if constexpr (P)
                t.e[r] = make_elem(k, p < count ? p : kPadRank);
            else
                t.k[r] = k;
        }
    }
    small_sort(t, lds[0], lds[1], wave, lane);
    // samples: the first and last key of every 64-key block and of the tile
    const uint32_t p0 = N * tid;
    if (src.out_smp.f != nullptr && (tid / 4) * kLine < count) {
        const uint64_t gpos = src.pos(blockIdx.x);
        const uint64_t b = gpos / kLine + tid / 4;
        if (tid % 4 == 0)
            src.out_smp.f[b] = key_of(t, 0);
        if (tid % 4 == 3)
            src.out_smp.l[b] = key_of(t, N - 1);
        if (src.out_smp.cf != nullptr && tid == 0)
            src.out_smp.cf[gpos / kTile] = key_of(t, 0);
        if (src.out_smp.cf != nullptr && tid == kSmallThreads - 1)
            src.out_smp.cl[gpos / kTile] = key_of(t, N - 1);
    }
    uint32_t ko[N], vo[N];
    if constexpr (P) {
        // values through LDS, by rank (the second buffer is free since the last barrier)
#pragma unroll
        for (int r = 0; r < N; ++r)
            lds[1][kSmallThreads * r + tid] = vals[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < N; ++r)
            vo[r] = lds[1][elem_rank(t.e[r]) & (kTile - 1)];  // padding reads some value, never stored
    }
#pragma unroll
    for (int r = 0; r < N; ++r) {
        ko[r] = key_of(t, r);
        if constexpr (Src::kMapped)
            ko[r] = map_key(ko[r], src.out_map.sign, src.out_map.rest, src.out_map.inverse);
    }
    if (p0 + N <= count) {
        Quad *kd = reinterpret_cast<Quad *>(it.kd + p0);
#pragma unroll
        for (int q = 0; q < N / 4; ++q)
            kd[q] = Quad{ko[4 * q], ko[4 * q + 1], ko[4 * q + 2], ko[4 * q + 3]};
        if constexpr (P) {
            Quad *vd = reinterpret_cast<Quad *>(it.vd + p0);
#pragma unroll
            for (int q = 0; q < N / 4; ++q)
                vd[q] = Quad{vo[4 * q], vo[4 * q + 1], vo[4 * q + 2], vo[4 * q + 3]};
        }
    } else {
#pragma unroll
        for (int r = 0; r < N; ++r)
            if (p0 + r < count) {
                it.kd[p0 + r] = ko[r];
                if constexpr (P)
                    it.vd[p0 + r] = vo[r];
            }
    }
}

// ----------------------------------------------------- merge by ranks
//
// A pass merges groups of `fan` (at most 16) consecutive runs of `run` keys (a
// multiple of 4096).  An element's place in its group is its index in its own
// run plus, for every other run, the number of elements there that precede
// it: those not above it in earlier runs, those below it in later runs (the
// stable order, so values just move along with their keys).  A work-group
// takes 256 consecutive elements of one run; the samples of the input bound
// the stretch of every other run that their ranks lie in, the stretches are
// staged in LDS (about 320 keys of each run where the runs interleave evenly),
// and every element searches each of them there.  Where the stretches do not
// fit, the searches read the runs themselves.  Every element costs (fan - 1)
// searches of about nine steps, so this is for sorts that leave the chip
// nearly empty: at 2^16 keys one launch of 11 us replaces four binary passes of
// 7 us, at 300,000 pairs two of 17 us replace three four-way passes and a binary
// one (113 us).  The searches read LDS words that depend on the data, so these
// reads, unlike the networks' exchanges, do have bank conflicts: 0.26 cycles per
// LDS instruction at 2^16 keys, 0.16 to 0.18 at 300,007 pairs.
constexpr uint32_t kRankMaxFan = 16;
constexpr uint32_t kRankChunk = 256;
constexpr uint32_t kRankStage = 6144;                      // staged words: 24 KiB
constexpr uint64_t kRankMaxRun = 32 * 64 * (uint64_t)kLine;  // two levels of 64 and 32 samples

struct RankSrc {
    const uint32_t *ksrc, *vsrc;
    uint32_t *kdst, *vdst;
    uint64_t n, run;
    uint32_t fan;
    const uint32_t *in_f;  // first key of every 64-key block of the input
    uint32_t *out_f;       // the same of the output, or nullptr
    KeyMap out_map;
};

// Lower bounds in B sorted runs of m[j] keys at once: how many keys are not
// above limit[j].  read(j, i) gives word i counted from one before run j's first
// key (so that i = 0, the word before it, is read and ignored where a run has
// no step left), and the steps are the same in every lane.  A step is three VALU
// instructions and one read per run.
template <int B, class Read>
__device__ __forceinline__ void rank_in_runs(const uint32_t (&limit)[B], const uint32_t (&m)[B], const Read &read,
                                             uint32_t (&at)[B])
{
    uint32_t len[B], most = 0;
#pragma unroll
    for (int j = 0; j < B; ++j) {
        at[j] = 0;
        len[j] = m[j];
        most = len[j] > most ? len[j] : most;
    }
    // halves while any run has more than one key left, then the last key
    for (bool end = false; !end; most -= most / 2) {
        end = most <= 1;
        uint32_t k[B], to[B];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const uint32_t half = end ? len[j] : len[j] / 2;
            to[j] = at[j] + half;
            len[j] -= half;
            k[j] = read(j, to[j]);
        }
#pragma unroll
        for (int j = 0; j < B; ++j)
            at[j] = k[j] <= limit[j] ? to[j] : at[j];
    }
}

template <bool P, bool MAP>
__global__ __launch_bounds__(kRankChunk) void k_rank_merge(RankSrc src)
{
    __shared__ uint32_t stage[1 + kRankStage];  // word 0 stands before the first run
    __shared__ uint32_t lo_s[kRankMaxFan], cnt_s[kRankMaxFan];
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    // one row of the grid per run, a column per chunk; sizes fit 32 bits
    const uint32_t n = (uint32_t)src.n, run = (uint32_t)src.run;
    const uint32_t rid = blockIdx.y, own = rid % src.fan;
    const uint32_t gstart = (rid - own) * run, left = n - gstart;
    const uint32_t in_run = blockIdx.x * kRankChunk;
    auto run_len = [&](uint32_t r) {  // of run r of the group (0 past its end)
        const uint32_t rest = left > r * run ? left - r * run : 0;
        return rest < run ? rest : run;
    };
    const uint32_t own_len = run_len(own);
    if (in_run >= own_len)
        return;  // the last run is shorter
    uint32_t runs = 1;
    while (runs < src.fan && runs * run < left)
        ++runs;
    const uint32_t count = own_len - in_run < kRankChunk ? own_len - in_run : kRankChunk;
    const uint32_t *K = src.ksrc + gstart;
    const uint32_t pos = own * run + in_run;  // in the group
    const uint32_t mine = pos + (tid < count ? tid : count - 1);
    const uint32_t x = K[mine];
    uint32_t v = 0;
    if constexpr (P)
        v = src.vsrc[gstart + mine];
    // the stretch of run r that the ranks of this chunk lie in, from its samples:
    // wave w bounds runs w, w + 4, ..., all loads of a level in flight at once
    // (a run that is not there, and the chunk's own, read some sample and drop it)
    constexpr int Q = (int)(kRankMaxFan / kSmallWaves);
    uint32_t S[Q], a[Q], a2[Q], b0[Q], b1[Q];
    const uint32_t *f[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint32_t r = wave + kSmallWaves * q;
        S[q] = r < runs && r != own ? (run_len(r) + kLine - 1) / kLine : 0;
        f[q] = src.in_f + (gstart + (S[q] ? r : own) * run) / kLine;
        const uint32_t i = lane * ((S[q] + kWave - 1) / kWave);  // every step-th sample; step at most 32
        a[q] = f[q][i < S[q] ? i : 0];
    }
    const uint32_t first = K[pos], last = K[pos + count - 1];
    __builtin_amdgcn_sched_barrier(0);
    auto precedes = [&](int q, uint32_t k, uint32_t y) { return wave + kSmallWaves * q < own ? k <= y : k < y; };
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint32_t step = (S[q] + kWave - 1) / kWave;
        const bool in = lane * step < S[q];
        b0[q] = __popcll(ballot(in && precedes(q, a[q], first)));
        b1[q] = __popcll(ballot(in && precedes(q, a[q], last)));
        // samples after the last one that precedes: lanes 0..31 for the first
        // key of the chunk, 32..63 for its last
        const uint32_t c = lane < 32 ? b0[q] : b1[q], i = (c - 1) * step + 1 + (lane & 31);
        const bool in2 = c != 0 && (lane & 31) + 1 < step && i < S[q];
        a2[q] = f[q][in2 ? i : 0];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint32_t r = wave + kSmallWaves * q, step = (S[q] + kWave - 1) / kWave;
        const uint32_t c = lane < 32 ? b0[q] : b1[q], i = (c - 1) * step + 1 + (lane & 31);
        const bool in2 = c != 0 && (lane & 31) + 1 < step && i < S[q];
        const uint64_t more = ballot(in2 && precedes(q, a2[q], lane < 32 ? first : last));
        const uint32_t m0 = b0[q] ? (b0[q] - 1) * step + 1 + __popc((uint32_t)more) : 0;
        const uint32_t m1 = b1[q] ? (b1[q] - 1) * step + 1 + __popc((uint32_t)(more >> 32)) : 0;
        // m samples precede: the rank is above 64 (m - 1) and at most 64 m
        const uint32_t len = S[q] ? run_len(r) : 0;
        const uint32_t lo = m0 ? kLine * (m0 - 1) + 1 : 0, hi = m1 * kLine < len ? m1 * kLine : len;
        if (lane == 0) {
            lo_s[r] = lo;
            cnt_s[r] = hi > lo ? hi - lo : 0;
        }
    }
    __syncthreads();
    uint32_t lo[kRankMaxFan], cnt[kRankMaxFan], off[kRankMaxFan], total = 0;
#pragma unroll
    for (int r = 0; r < (int)kRankMaxFan; ++r) {
        lo[r] = uniform(lo_s[r]);
        cnt[r] = uniform(cnt_s[r]);
        off[r] = total;
        total += cnt[r];
    }
    uint32_t place = in_run + tid;
    if (total <= kRankStage) {
        // direct global-to-LDS loads, all of a wave's runs in flight at once
#pragma unroll
        for (int q = 0; q < (int)(kRankMaxFan / kSmallWaves); ++q) {
            const uint32_t r = wave + kSmallWaves * q;
            const uint32_t c = uniform(cnt_s[r]);
            uint32_t o = 1;
#pragma unroll
            for (int i = 0; i < (int)kRankMaxFan; ++i)
                o += (uint32_t)i < r ? cnt[i] : 0;
            const uint32_t *s = K + r * run + uniform(lo_s[r]);
            for (uint32_t i = 0; i < c; i += kWave)
                if (i + lane < c)
                    __builtin_amdgcn_global_load_lds((global_cvoid *)(s + i + lane), (lds_void *)(stage + o + i), 4, 0, 0);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
    auto rank_from = [&](auto first_run, auto width) {
        constexpr int b = decltype(first_run)::value, B = decltype(width)::value;
        uint32_t m[B], at[B], limit[B];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            m[j] = cnt[b + j];
            // keys below x are those not above x - 1 (none when x is 0, below)
            limit[j] = (uint32_t)(b + j) < own ? x : x - 1;
        }
        if (total <= kRankStage)
            rank_in_runs<B>(limit, m, [&](int j, uint32_t i) { return stage[off[b + j] + i]; }, at);
        else
            rank_in_runs<B>(limit, m,
                            [&](int j, uint32_t i) {
                                return K[(m[j] ? (b + j) * run + lo[b + j] : 0) + (i ? i - 1 : 0)];
                            },
                            at);
#pragma unroll
        for (int j = 0; j < B; ++j)
            place += lo[b + j] + (x == 0 && (uint32_t)(b + j) > own ? 0 : at[j]);
    };
    // searches in flight per lane: eight, or four for the last few runs
    using I0 = std::integral_constant<int, 0>;
    using I4 = std::integral_constant<int, 4>;
    using I8 = std::integral_constant<int, 8>;
    if (runs <= 4) {
        rank_from(I0(), I4());
    } else {
        rank_from(I0(), I8());
        if (runs > 12)
            rank_from(I8(), I8());
        else if (runs > 8)
            rank_from(I8(), I4());
    }
    if (tid >= count)
        return;
    const uint32_t p = gstart + place;
    if (src.out_f != nullptr && p % kLine == 0)
        src.out_f[p / kLine] = x;
    uint32_t out = x;
    if constexpr (MAP)
        out = map_key(x, src.out_map.sign, src.out_map.rest, src.out_map.inverse);
    src.kdst[p] = out;
    if constexpr (P)
        src.vdst[p] = v;
}

}  // namespace bcf
