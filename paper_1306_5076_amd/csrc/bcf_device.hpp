// Device building blocks of the bank-conflict-free sort for gfx950 (CDNA4, wave64).
//
// The paper (Sitchinava & Weichert, Sec. 2.1) views a block of shared memory as
// a matrix whose rows are the memory banks, filled column-major, and processes
// it so that every thread of a warp owns one bank row; a conflict-free
// transposition turns columns into rows.  Its sort (Sec. 3.1) keeps one line of
// the w x w tile in registers per thread (Sec. 3.3, "use of registers") and
// sorts lines with Batcher's odd-even merge sort.
//
// Re-derived for gfx950 (measured: 32 banks x 4 bytes; a wave64 b32 LDS
// instruction is serviced as two independent 32-lane halves):
//   * a tile is a 64 x 64 matrix of keys, w = 64 = wave width, so one wave owns
//     w^2 = 4096 keys, 64 per lane, held in registers with compile-time indices;
//   * two register layouts of tile position p in [0, 4096):
//       STRIDED  lane = p mod 64, register = p / 64   (global loads/stores are
//                coalesced: register r of all lanes is 64 consecutive keys)
//       BLOCKED  lane = p / 64,   register = p mod 64 (lane owns a run of 64)
//   * switching layouts goes through LDS with four pad words per 64
//     (address = p + 4 (p/64)): STRIDED accesses are 4-byte reads and writes
//     of word 68r + lane, so every 32-lane half touches 32 distinct banks;
//     BLOCKED accesses move four consecutive registers at once, 16 bytes at
//     word 68 lane + r (r a multiple of 4): lane l's first bank is
//     4l + r mod 32, so the 8 consecutive lanes that a write of 16 bytes
//     services together cover the 32 banks once, and mod 64 the 16 lanes that
//     a read services together (lanes of every value mod 16) the 64 banks that
//     reads have.  The lane-dependent part of an address is a base register
//     and the register-dependent part an immediate offset;
//   * compare-exchanges only ever happen between two registers of one lane, so
//     the sorting networks themselves issue no LDS traffic at all.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bcf {

constexpr int kWave = 64;              // lanes per wavefront (w)
constexpr int kLine = 64;              // keys per lane (one line of the w x w tile)
constexpr int kTile = kWave * kLine;   // 4096 keys per wave tile (w^2)
constexpr int kLdsPad = 4;                   // pad words per 64-word LDS row
constexpr int kLdsStride = kLine + kLdsPad;  // 68 words per LDS row
constexpr int kLdsWords = kWave * kLdsStride;

constexpr uint32_t kMaxKey = 0xFFFFFFFFu;

// A wave's tile in registers.  Keys only: one 32-bit key per position.
//
// Key/value pairs: one 64-bit element per position that orders by (key,
// rank), where the rank is the element's position in the input order of the
// tile; comparing ranks on equal keys makes every network stable.  The
// element is a double in [1, 2) whose mantissa holds key * 2^15 + rank: such
// doubles are finite, normal and positive, so they order exactly as that
// 47-bit integer, and a compare-exchange is one v_min_f64 and one v_max_f64
// (full-rate on CDNA4), the same two instructions as for keys.  Values do not
// travel through the networks: after the last network the rank names the
// input position whose value goes with the key, the value is fetched by it
// (from LDS in the block sort, from global memory in a merge) and the element
// is repacked as key (high half) and value (low half) for the store.
template <bool PAIRS>
struct Lines {
    uint32_t k[kLine];
};
template <>
struct Lines<true> {
    double e[kLine];
};

// Unsigned 64-bit keys: one key per position in a register pair, compared as
// integers (no values, no ranks: equal keys are indistinguishable).
struct Lines64 {
    uint64_t e[kLine];
};
constexpr uint64_t kMaxKey64 = ~0ull;

constexpr uint32_t kRankBits = 15;                    // group tiles of up to 32768 positions
constexpr uint32_t kPadRank = (1u << kRankBits) - 1;  // rank of padding (never a real rank)
constexpr int kRankShift = 52 - 32 - (int)kRankBits;  // payload in mantissa bits 51 .. 5
constexpr uint64_t kElemOne = 0x3FF0000000000000ull;  // sign and exponent of 1.0
constexpr uint64_t kPayloadMask = ((1ull << (32 + kRankBits)) - 1) << kRankShift;

__device__ __forceinline__ uint64_t bits_of(double x) { return __builtin_bit_cast(uint64_t, x); }
__device__ __forceinline__ double elem_of(uint64_t b) { return __builtin_bit_cast(double, b); }

__device__ __forceinline__ double make_elem(uint32_t key, uint32_t rank)
{
    return elem_of(kElemOne | ((uint64_t)key << (kRankShift + kRankBits)) | ((uint64_t)rank << kRankShift));
}
__device__ __forceinline__ uint32_t elem_key(double e) { return (uint32_t)(bits_of(e) >> (kRankShift + kRankBits)); }
__device__ __forceinline__ uint32_t elem_rank(double e) { return (uint32_t)(bits_of(e) >> kRankShift) & kPadRank; }

// After the value step: key in the high half, value in the low half.
__device__ __forceinline__ double make_out(uint32_t key, uint32_t value)
{
    return elem_of(((uint64_t)key << 32) | value);
}
__device__ __forceinline__ uint32_t out_key(double e) { return (uint32_t)(bits_of(e) >> 32); }
__device__ __forceinline__ uint32_t out_value(double e) { return (uint32_t)bits_of(e); }

// Key of register r of a tile that is still in element form.
template <bool P>
__device__ __forceinline__ uint32_t key_of(const Lines<P> &t, int r)
{
    if constexpr (P)
        return elem_key(t.e[r]);
    else
        return t.k[r];
}

// ---------------------------------------------------------------- comparators

// The register-local networks compile for the host too, where they can be run
// on every 0-1 input: they are minima and maxima only, so by the 0-1 principle
// that decides them for all keys.
#define BCF_HD __host__ __device__ __forceinline__

BCF_HD uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }
BCF_HD uint32_t umax(uint32_t a, uint32_t b) { return a < b ? b : a; }

// Put the smaller element in register a, the larger in register b.
template <bool P>
BCF_HD void cx(Lines<P> &t, int a, int b)
{
    if constexpr (!P) {
        const uint32_t x = t.k[a], y = t.k[b];
        t.k[a] = umin(x, y);
        t.k[b] = umax(x, y);
    } else {
        const double x = t.e[a], y = t.e[b];
        t.e[a] = __builtin_fmin(x, y);
        t.e[b] = __builtin_fmax(x, y);
    }
}

// 64-bit keys: one unsigned 64-bit compare and four 32-bit selects.
BCF_HD void cx(Lines64 &t, int a, int b)
{
    const uint64_t x = t.e[a], y = t.e[b];
    const bool lt = x < y;
    t.e[a] = lt ? x : y;
    t.e[b] = lt ? y : x;
}

// Reverse the order of every element of a lane when `bit` is 1: the key (or
// the element's payload) is replaced by its bitwise complement, an
// order-reversing bijection, so an ascending network run on complemented data
// sorts descending.  Used where
// the direction of a merge depends on the lane (BLOCKED layout).
template <bool P>
__device__ __forceinline__ void flip(Lines<P> &t, uint32_t bit)
{
    const uint32_t m = 0u - (bit & 1u);
#pragma unroll
    for (int r = 0; r < kLine; ++r) {
        if constexpr (P)  // complement the payload only: the element stays in [1, 2)
            t.e[r] = elem_of(bits_of(t.e[r]) ^ (kPayloadMask & ((uint64_t)m << 32 | m)));
        else
            t.k[r] ^= m;
    }
}

__device__ __forceinline__ void flip(Lines64 &t, uint32_t bit)
{
    const uint64_t m = 0ull - (uint64_t)(bit & 1u);
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        t.e[r] ^= m;
}

// ---------------------------------------------------- register-local networks
//
// Written once for any line type L (Lines<false>, Lines<true>, Lines64): the
// compare-exchange cx(t, a, b) is chosen by overload.

// One bitonic half-cleaner step at register distance D: registers r and r+D
// (r with bit D clear) are compare-exchanged, ascending, or descending where
// register bit DB of r is set (DB < 0: ascending everywhere).
template <int D, int DB, class L>
BCF_HD void half_clean_step_lines(L &t)
{
#pragma unroll
    for (int r = 0; r < kLine; ++r) {
        if (r & D)
            continue;
        if (DB >= 0 && ((r >> (DB < 0 ? 0 : DB)) & 1))
            cx(t, r + D, r);
        else
            cx(t, r, r + D);
    }
}

// Three-input minimum, median and maximum of u32 keys: one VALU instruction
// each (v_min3_u32, v_med3_u32, v_max3_u32), at the rate of v_min_u32 from two
// waves per SIMD on.  The compiler forms them only when no inner minimum or
// maximum is shared, so their users below pass the operands in an order that
// pairs them differently in each call.
BCF_HD uint32_t min3(uint32_t a, uint32_t b, uint32_t c) { return umin(umin(a, b), c); }
BCF_HD uint32_t max3(uint32_t a, uint32_t b, uint32_t c) { return umax(umax(a, b), c); }
BCF_HD uint32_t med3(uint32_t a, uint32_t b, uint32_t c) { return umax(umin(a, b), umin(umax(a, b), c)); }

// Two half-cleaner steps at once, distances D and D/2, on u32 keys.  With
// (a, b, c, d) at r, r + D/2, r + D, r + 3D/2 the first step pairs (a, c) and
// (b, d).  (a, b, c, d) is bitonic, so both minima of the first step are at
// most both maxima: with p = min(a, c) <= max(b, d) the second step's outputs
// min(p, min(b, d)) and max(p, min(b, d)) are min3(p, b, d) and
// med3(p, b, d), and likewise for P = max(a, c): six instructions in place of
// eight.  Measured on the six steps of 64 registers: 506 ns per wave against
// 656 ns at four waves per SIMD (596 against 707 ns at one).
template <int D, int DB>
BCF_HD void half_clean_pair(Lines<false> &t)
{
    constexpr int E = D / 2;
#pragma unroll
    for (int r = 0; r < kLine; ++r) {
        if (r & (D | E))
            continue;
        const uint32_t a = t.k[r], b = t.k[r + E], c = t.k[r + D], d = t.k[r + D + E];
        const uint32_t p = umin(a, c), q = umax(a, c);
        const bool desc = DB >= 0 && ((r >> (DB < 0 ? 0 : DB)) & 1);
        t.k[desc ? r + D + E : r] = min3(p, d, b);
        t.k[desc ? r + D : r + E] = med3(b, d, p);
        t.k[desc ? r + E : r + D] = med3(b, d, q);
        t.k[desc ? r : r + D + E] = max3(q, d, b);
    }
}

// Half-cleaner cascade D, D/2, ..., 1: sorts every aligned group of 2D
// registers that holds a bitonic sequence.
template <int D, int DB, class L>
BCF_HD void half_clean_lines(L &t)
{
    half_clean_step_lines<D, DB>(t);
    if constexpr (D > 1)
        half_clean_lines<D / 2, DB>(t);
}
template <int D, int DB>
BCF_HD void half_clean_lines(Lines<false> &t)
{
    if constexpr (D > 1) {
        half_clean_pair<D, DB>(t);
        if constexpr (D > 2)
            half_clean_lines<D / 4, DB>(t);
    } else {
        half_clean_step_lines<D, DB>(t);
    }
}

// Batcher's odd-even merge of registers LO..HI (inclusive) whose two halves
// are sorted, considering every R-th register (Batcher 1968; the recursive
// formulation in Knuth, TAOCP vol. 3, Sec. 5.3.4).
template <int LO, int HI, int R, class L>
BCF_HD void oe_merge_lines(L &t)
{
    constexpr int STEP = 2 * R;
    if constexpr (STEP < HI - LO) {
        oe_merge_lines<LO, HI, STEP>(t);
        oe_merge_lines<LO + R, HI, STEP>(t);
#pragma unroll
        for (int i = LO + R; i < HI - R; i += STEP)
            cx(t, i, i + R);
    } else {
        cx(t, LO, LO + R);
    }
}

// Batcher's odd-even merge sort of registers LO..HI (inclusive), ascending:
// the per-thread line sort of the paper (Sec. 3.1; 543 comparators for 64).
template <int LO, int HI, class L>
BCF_HD void oe_sort_lines(L &t)
{
    if constexpr (HI - LO >= 1) {
        constexpr int MID = LO + (HI - LO) / 2;
        oe_sort_lines<LO, MID>(t);
        oe_sort_lines<MID + 1, HI>(t);
        oe_merge_lines<LO, HI, 1>(t);
    }
}

// The same merge on u32 keys, written step by step (distances N/2, N/4, ...,
// 1; step d < N/2 pairs i and i + d where i / d is odd) so that two steps
// share three-input instructions.
//
// The first two steps of N = HI - LO + 1 registers merge (a <= b) with
// (c <= d), a quarter apart: the outputs are min(a, c), then with y = min(b, d)
// >= min(a, c) the second comparator's min and max of (max(a, c), y) are
// med3(a, c, y) and max3(a, c, y), then max(b, d): five instructions for six.
template <int LO, int N>
BCF_HD void oe_first_pair(Lines<false> &t)
{
    constexpr int Q = N / 4;
#pragma unroll
    for (int i = LO; i < LO + Q; ++i) {
        const uint32_t a = t.k[i], b = t.k[i + Q], c = t.k[i + 2 * Q], d = t.k[i + 3 * Q];
        const uint32_t y = umin(b, d);
        t.k[i] = umin(a, c);
        t.k[i + 2 * Q] = max3(a, y, c);
        t.k[i + Q] = med3(c, y, a);
        t.k[i + 3 * Q] = umax(b, d);
    }
}

// One step at distance D.
template <int LO, int N, int D>
BCF_HD void oe_single(Lines<false> &t)
{
#pragma unroll
    for (int i = 0; i + D < N; ++i)
        if (D == N / 2 ? i < D : (i / D) % 2 == 1)
            cx(t, LO + i, LO + i + D);
}

// Two later steps at distances 2D and D (2D < N/2).  Step 2D leaves
// lo = min(e, f) and hi = max(e, f) at i and i + 2D; step D pairs every hi
// (and the first step's unpaired registers) with the next register's z, and
// lo <= z there (the evens and odds are sorted by then), so min(hi, z) =
// med3(e, f, z) and max(hi, z) = max3(e, f, z): hi itself is never computed.
template <int LO, int N, int D>
BCF_HD void oe_later_pair(Lines<false> &t)
{
#pragma unroll
    for (int o = 0; o < D; ++o) {  // registers o, o + D, o + 2D, ...: position q of the chain
        constexpr int M = N / D;
        uint32_t e[M];
#pragma unroll
        for (int q = 0; q < M; ++q)
            e[q] = t.k[LO + o + D * q];
        // after step 2D, position q holds lo of (q, q + 2) when q % 4 is 2 or
        // 3 (q + 2 < M), hi of (q - 2, q) when q % 4 is 0 or 1 (q >= 4)
        auto first = [&](int q) { return (q % 4 >= 2 && q + 2 < M) ? umin(e[q], e[q + 2]) : e[q]; };
#pragma unroll
        for (int q = 1; q + 1 < M; q += 2) {
            // step D pairs q and q + 1: one of them is a lo (or unpaired), the
            // other a hi (or unpaired)
            const int h = q % 4 == 1 ? q : q + 1;      // the hi side
            const int w = q % 4 == 1 ? q + 1 : q;      // the lo side
            const uint32_t z = first(w);
            uint32_t lo, hi;
            if (h >= 4) {
                lo = med3(e[h], z, e[h - 2]);
                hi = max3(e[h - 2], z, e[h]);
            } else {
                lo = umin(e[h], z);
                hi = umax(e[h], z);
            }
            t.k[LO + o + D * q] = lo;
            t.k[LO + o + D * (q + 1)] = hi;
        }
    }
}

// Steps D, D/2, ... of the merge after the first ones, two at a time.
template <int LO, int N, int D>
BCF_HD void oe_later_steps(Lines<false> &t)
{
    if constexpr (D >= 2) {
        oe_later_pair<LO, N, D / 2>(t);
        oe_later_steps<LO, N, D / 4>(t);
    }
}

template <int LO, int N>
BCF_HD void oe_merge_keys(Lines<false> &t)
{
    // log2(N) steps: an even number starts with the first pair, an odd one
    // with a single step (distance N/2), then pairs
    if constexpr (N == 16 || N == 64) {
        oe_first_pair<LO, N>(t);
        oe_later_steps<LO, N, N / 8>(t);
    } else {
        static_assert(N == 8 || N == 32, "merge sizes");
        oe_single<LO, N, N / 2>(t);
        oe_later_steps<LO, N, N / 4>(t);
    }
}

// Four registers sorted by inserting the fourth into the sorted first three:
// seven instructions for the ten of five comparators.
template <int LO>
BCF_HD void sort4(Lines<false> &t)
{
    const uint32_t a = t.k[LO], b = t.k[LO + 1], c = t.k[LO + 2], d = t.k[LO + 3];
    const uint32_t x = min3(a, c, b), z = max3(a, c, b), y = med3(b, c, a);
    t.k[LO] = umin(x, d);
    t.k[LO + 3] = umax(z, d);
    t.k[LO + 1] = med3(x, y, d);
    t.k[LO + 2] = med3(y, z, d);
}

// The line sort of u32 keys: sorted fours, then odd-even merges.  868
// instructions for 64 keys in place of the 1086 of 543 comparators.
template <int LO, int HI>
BCF_HD void oe_sort_lines(Lines<false> &t)
{
    constexpr int N = HI - LO + 1;
    static_assert(N == 4 || N == 8 || N == 16 || N == 32 || N == 64, "line sizes");
    if constexpr (N == 4) {
        sort4<LO>(t);
    } else {
        oe_sort_lines<LO, LO + N / 2 - 1>(t);
        oe_sort_lines<LO + N / 2, HI>(t);
        oe_merge_keys<LO, N>(t);
    }
}

// The same networks for the 32-bit element kinds, named by the pairs flag.
template <int D, int DB, bool P>
__device__ __forceinline__ void half_clean(Lines<P> &t)
{
    half_clean_lines<D, DB>(t);
}
template <int LO, int HI, bool P>
__device__ __forceinline__ void oe_sort(Lines<P> &t)
{
    oe_sort_lines<LO, HI>(t);
}

// ------------------------------------------------------------ LDS transposes

// Orders this wave's LDS accesses in the compiler: a wave's LDS instructions
// execute in issue order, so no hardware wait is needed between a lane's
// write and another lane's later read of the same word.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// x[r] -> w[S*r] for r = 0..63.  With S = 1 (the BLOCKED side: a lane's
// registers are consecutive words and the row starts 16-byte aligned) the
// compiler merges every four registers into one 16-byte store.
template <int S>
__device__ __forceinline__ void lds_put(uint32_t *w, const uint32_t (&x)[kLine])
{
    if constexpr (S == 1)
        w = static_cast<uint32_t *>(__builtin_assume_aligned(w, 16));
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        w[S * r] = x[r];
}

// x[r] <- rd[S*r] for r = 0..63 (S = 1: 16-byte loads).
template <int S>
__device__ __forceinline__ void lds_get(uint32_t (&x)[kLine], const uint32_t *rd)
{
    if constexpr (S == 1)
        rd = static_cast<const uint32_t *>(__builtin_assume_aligned(rd, 16));
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        x[r] = rd[S * r];
}

// x[r] -> lds[wbase + WS*r], then x[r] <- lds[rbase + RS*r].
template <int WS, int RS>
__device__ __forceinline__ void exchange(uint32_t (&x)[kLine], uint32_t *lds, uint32_t wbase,
                                         uint32_t rbase)
{
    lds_put<WS>(lds + wbase, x);
    wave_lds_fence();
    lds_get<RS>(x, lds + rbase);
    wave_lds_fence();
}

// The 32-bit halves of 64-bit elements.
__device__ __forceinline__ void split_halves(const double (&x)[kLine], uint32_t (&hi)[kLine], uint32_t (&lo)[kLine])
{
#pragma unroll
    for (int r = 0; r < kLine; ++r) {
        hi[r] = (uint32_t)(bits_of(x[r]) >> 32);
        lo[r] = (uint32_t)bits_of(x[r]);
    }
}

__device__ __forceinline__ void split_halves(const uint64_t (&x)[kLine], uint32_t (&hi)[kLine], uint32_t (&lo)[kLine])
{
#pragma unroll
    for (int r = 0; r < kLine; ++r) {
        hi[r] = (uint32_t)(x[r] >> 32);
        lo[r] = (uint32_t)x[r];
    }
}
__device__ __forceinline__ void join_halves(double (&x)[kLine], const uint32_t (&hi)[kLine], const uint32_t (&lo)[kLine])
{
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        x[r] = elem_of(((uint64_t)hi[r] << 32) | lo[r]);
}
__device__ __forceinline__ void join_halves(uint64_t (&x)[kLine], const uint32_t (&hi)[kLine],
                                            const uint32_t (&lo)[kLine])
{
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        x[r] = ((uint64_t)hi[r] << 32) | lo[r];
}

// The same for 64-bit elements, one 32-bit half at a time (each half keeps the
// conflict-free word pattern of the 32-bit exchange).
template <int WS, int RS>
__device__ __forceinline__ void exchange(double (&x)[kLine], uint32_t *lds, uint32_t wbase, uint32_t rbase)
{
    uint32_t hi[kLine], lo[kLine];
    split_halves(x, hi, lo);
    exchange<WS, RS>(hi, lds, wbase, rbase);
    exchange<WS, RS>(lo, lds, wbase, rbase);
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        x[r] = elem_of(((uint64_t)hi[r] << 32) | lo[r]);
}

// The same for 64-bit keys.
template <int WS, int RS>
__device__ __forceinline__ void exchange(uint64_t (&x)[kLine], uint32_t *lds, uint32_t wbase, uint32_t rbase)
{
    uint32_t hi[kLine], lo[kLine];
#pragma unroll
    for (int r = 0; r < kLine; ++r) {
        hi[r] = (uint32_t)(x[r] >> 32);
        lo[r] = (uint32_t)x[r];
    }
    exchange<WS, RS>(hi, lds, wbase, rbase);
    exchange<WS, RS>(lo, lds, wbase, rbase);
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        x[r] = ((uint64_t)hi[r] << 32) | lo[r];
}

__device__ __forceinline__ uint64_t (&elems(Lines64 &t))[kLine] { return t.e; }

template <bool P>
__device__ __forceinline__ auto &elems(Lines<P> &t)
{
    if constexpr (P)
        return t.e;
    else
        return t.k;
}

// STRIDED -> BLOCKED: write word 68r + lane, read word 68 lane + r.
template <class L>
__device__ __forceinline__ void to_blocked(L &t, uint32_t *lds, uint32_t lane)
{
    exchange<kLdsStride, 1>(elems(t), lds, lane, kLdsStride * lane);
}

// BLOCKED -> STRIDED: write word 68 lane + r, read word 68r + lane.  Afterwards
// LDS word 68q + r holds tile position 64q + r.
template <class L>
__device__ __forceinline__ void to_strided(L &t, uint32_t *lds, uint32_t lane)
{
    exchange<1, kLdsStride>(elems(t), lds, kLdsStride * lane, lane);
}

// ------------------------------------------ half-width transposes (9 KiB LDS)
//
// The same STRIDED <-> BLOCKED transposes with half the LDS: view the tile as
// the 64 x 64 matrix M[register][lane].  v_permlane32_swap on registers r and
// r + 32 (r < 32) exchanges the upper half-wave of register r with the lower
// half-wave of register r + 32, which swaps the off-diagonal 32 x 32 quadrants
// of M; afterwards each half-wave holds two 32 x 32 blocks (registers 0..31
// and 32..63) that only need transposing inside the half-wave.  Each block
// goes through a 32-row LDS matrix per half-wave (rows of 36 words), one
// block after the other, so a wave needs 2 x 32 x 36 words instead of
// 64 x 68.  Accesses stay conflict-free on the measured geometry: 4-byte
// writes / reads of word 36r + l' (32 consecutive words per half-wave), and
// 16-byte reads / writes of word 36l' + c, c a multiple of 4 (36 = 4 mod 32:
// 8 consecutive lanes cover the 32 banks of writes once, 16 lanes of every value
// mod 16 the 64 banks of reads).
constexpr int kHalfRows = 32;
constexpr int kHalfStride = 36;
constexpr int kHalfLdsWords = 2 * kHalfRows * kHalfStride;  // per wave: 9 KiB

// Exchange the upper half-wave of register r with the lower half-wave of
// register r + 32, for r = 0..31.
__device__ __forceinline__ void swap_quadrants(uint32_t (&x)[kLine])
{
#pragma unroll
    for (int r = 0; r < kLine / 2; ++r) {
        const auto p = __builtin_amdgcn_permlane32_swap(x[r], x[r + kLine / 2], false, false);
        x[r] = p[0];
        x[r + kLine / 2] = p[1];
    }
}

// This half-wave's 32 x 36-word LDS matrix.
__device__ __forceinline__ uint32_t *half_matrix(uint32_t *lds, uint32_t lane)
{
    return lds + (lane >> 5) * (kHalfRows * kHalfStride);
}

// Transpose the 32 x 32 block in registers R0..R0+31 inside each half-wave:
// the STRIDED side (register r, lane l') at word 36r + l', the BLOCKED side
// (lane l', register c) at word 36l' + c.  S2B: STRIDED side in, BLOCKED
// side out; else the reverse.
template <int R0, bool S2B>
__device__ __forceinline__ void half_block_transpose(uint32_t (&x)[kLine], uint32_t *lds, uint32_t lane)
{
    uint32_t *m = half_matrix(lds, lane);
    const uint32_t l = lane & 31;
    uint32_t *row = static_cast<uint32_t *>(__builtin_assume_aligned(m + kHalfStride * l, 16));
    if constexpr (S2B) {
#pragma unroll
        for (int r = 0; r < kHalfRows; ++r)
            m[kHalfStride * r + l] = x[R0 + r];
        wave_lds_fence();
#pragma unroll
        for (int c = 0; c < kHalfRows; ++c)
            x[R0 + c] = row[c];
    } else {
#pragma unroll
        for (int c = 0; c < kHalfRows; ++c)
            row[c] = x[R0 + c];
        wave_lds_fence();
#pragma unroll
        for (int r = 0; r < kHalfRows; ++r)
            x[R0 + r] = m[kHalfStride * r + l];
    }
    wave_lds_fence();
}

// STRIDED -> BLOCKED (keys) through the half-width matrices.
__device__ __forceinline__ void to_blocked_half(Lines<false> &t, uint32_t *lds, uint32_t lane)
{
    swap_quadrants(t.k);
    half_block_transpose<0, true>(t.k, lds, lane);
    half_block_transpose<kLine / 2, true>(t.k, lds, lane);
}

// BLOCKED -> STRIDED (keys) through the half-width matrices.
__device__ __forceinline__ void to_strided_half(Lines<false> &t, uint32_t *lds, uint32_t lane)
{
    half_block_transpose<0, false>(t.k, lds, lane);
    half_block_transpose<kLine / 2, false>(t.k, lds, lane);
    swap_quadrants(t.k);
}

// The same two transposes for 64-bit elements, one 32-bit half after the
// other through the same matrices.
template <class E>
__device__ __forceinline__ void to_blocked_half_wide(E (&x)[kLine], uint32_t *lds, uint32_t lane)
{
    uint32_t hi[kLine], lo[kLine];
    split_halves(x, hi, lo);
    swap_quadrants(hi);
    half_block_transpose<0, true>(hi, lds, lane);
    half_block_transpose<kLine / 2, true>(hi, lds, lane);
    swap_quadrants(lo);
    half_block_transpose<0, true>(lo, lds, lane);
    half_block_transpose<kLine / 2, true>(lo, lds, lane);
    join_halves(x, hi, lo);
}
template <class E>
__device__ __forceinline__ void to_strided_half_wide(E (&x)[kLine], uint32_t *lds, uint32_t lane)
{
    uint32_t hi[kLine], lo[kLine];
    split_halves(x, hi, lo);
    half_block_transpose<0, false>(hi, lds, lane);
    half_block_transpose<kLine / 2, false>(hi, lds, lane);
    swap_quadrants(hi);
    half_block_transpose<0, false>(lo, lds, lane);
    half_block_transpose<kLine / 2, false>(lo, lds, lane);
    swap_quadrants(lo);
    join_halves(x, hi, lo);
}
__device__ __forceinline__ void to_blocked_half(Lines<true> &t, uint32_t *lds, uint32_t lane)
{
    to_blocked_half_wide(t.e, lds, lane);
}
__device__ __forceinline__ void to_strided_half(Lines<true> &t, uint32_t *lds, uint32_t lane)
{
    to_strided_half_wide(t.e, lds, lane);
}
__device__ __forceinline__ void to_blocked_half(Lines64 &t, uint32_t *lds, uint32_t lane)
{
    to_blocked_half_wide(t.e, lds, lane);
}
__device__ __forceinline__ void to_strided_half(Lines64 &t, uint32_t *lds, uint32_t lane)
{
    to_strided_half_wide(t.e, lds, lane);
}

// ------------------------------------------------------ group (multi-wave) sort
//
// NW waves of a work-group (NW = 2^LW) sort a group tile of NW * 4096 keys:
// every wave sorts its 4096-key sub-tile (odd waves descending, by
// complementing around the wave sort), then LW more bitonic rounds
// (J = 7 .. 6+LW) merge across waves.  Wave w holds group positions with
// bits 12.. equal to w.  A third layout brings the wave bits into registers:
//   CROSS  lane = p bits 0..5, wave = p bits 6..5+LW, register = p bits 6+LW..11+LW
// Round J: BLOCKED -> CROSS (shared LDS, barriers), stages on bits 5+J..6+LW
// in registers, CROSS -> STRIDED, stages on bits 5+LW..6, STRIDED -> BLOCKED
// (the wave's own LDS slice), stages on bits 5..0.  The LDS word of position
// p is p + 4 (p/64) in all three layouts, so every access keeps the 68-word
// rows of the single-wave transposes: lane-consecutive 4-byte accesses (CROSS,
// STRIDED) touch 32 distinct banks per 32-lane half, and BLOCKED accesses are
// 16-byte, four registers at a time, 8 lanes covering the 32 banks.

// x[r] -> lds[wbase + WS*r]; barrier; x[r] <- lds[rbase + RS*r]; barrier.
template <int WS, int RS>
__device__ __forceinline__ void group_exchange(uint32_t (&x)[kLine], uint32_t *lds, uint32_t wbase,
                                               uint32_t rbase)
{
    lds_put<WS>(lds + wbase, x);
    __syncthreads();
    lds_get<RS>(x, lds + rbase);
    __syncthreads();
}

// The same for 64-bit elements, one 32-bit half at a time.
template <int WS, int RS>
__device__ __forceinline__ void group_exchange(double (&x)[kLine], uint32_t *lds, uint32_t wbase, uint32_t rbase)
{
    uint32_t hi[kLine], lo[kLine];
    split_halves(x, hi, lo);
    group_exchange<WS, RS>(hi, lds, wbase, rbase);
    group_exchange<WS, RS>(lo, lds, wbase, rbase);
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        x[r] = elem_of(((uint64_t)hi[r] << 32) | lo[r]);
}

// The same for 64-bit keys.
template <int WS, int RS>
__device__ __forceinline__ void group_exchange(uint64_t (&x)[kLine], uint32_t *lds, uint32_t wbase, uint32_t rbase)
{
    uint32_t hi[kLine], lo[kLine];
#pragma unroll
    for (int r = 0; r < kLine; ++r) {
        hi[r] = (uint32_t)(x[r] >> 32);
        lo[r] = (uint32_t)x[r];
    }
    group_exchange<WS, RS>(hi, lds, wbase, rbase);
    group_exchange<WS, RS>(lo, lds, wbase, rbase);
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        x[r] = ((uint64_t)hi[r] << 32) | lo[r];
}

// BLOCKED p = 4096w + 64 lane + r  ->  CROSS p = lane + 64w + 64*NW*r
template <int NW, class L>
__device__ __forceinline__ void blocked_to_cross(L &t, uint32_t *lds, uint32_t lane, uint32_t wave)
{
    const uint32_t wb = kLdsStride * (kWave * wave + lane), rb = kLdsStride * wave + lane;
    group_exchange<1, kLdsStride * NW>(elems(t), lds, wb, rb);
}

// CROSS p = lane + 64w + 64*NW*r  ->  STRIDED p = 4096w + 64r + lane
template <int NW, class L>
__device__ __forceinline__ void cross_to_strided(L &t, uint32_t *lds, uint32_t lane, uint32_t wave)
{
    const uint32_t wb = kLdsStride * wave + lane, rb = kLdsStride * kWave * wave + lane;
    group_exchange<kLdsStride * NW, kLdsStride>(elems(t), lds, wb, rb);
}

constexpr int log2i(int x) { return x <= 1 ? 0 : 1 + log2i(x / 2); }

// Round J (7 .. 6+LW) of the group sort; on entry and exit the tile is
// BLOCKED and every run of 2^(6+J) positions is sorted, descending where bit
// 6+J is set (the last round sorts ascending).
template <int NW, int J, class L>
__device__ __forceinline__ void group_round(L &t, uint32_t *lds, uint32_t lane, uint32_t wave)
{
    constexpr int LW = log2i(NW);
    constexpr bool last = J == 6 + LW;
    blocked_to_cross<NW>(t, lds, lane, wave);
    // bits 5+J .. 6+LW = CROSS register bits J-1-LW .. 0; direction bit 6+J = register bit J-LW
    half_clean_lines<(1 << (J - 1 - LW)), (last ? -1 : J - LW)>(t);
    cross_to_strided<NW>(t, lds, lane, wave);
    // bits 5+LW .. 6 = STRIDED register bits LW-1 .. 0; direction bit 6+J = wave bit J-6
    if constexpr (!last)
        flip(t, wave >> (J - 6));
    half_clean_lines<(1 << (LW - 1)), -1>(t);
    to_blocked(t, lds + kLdsWords * wave, lane);
    half_clean_lines<kLine / 2, -1>(t);
    if constexpr (!last)
        flip(t, wave >> (J - 6));
}

// Rounds J .. 6 + log2(NW) of a group tile (any line type).
template <int NW, int J, class L>
__device__ __forceinline__ void group_rounds(L &t, uint32_t *lds, uint32_t lane, uint32_t wave)
{
    group_round<NW, J>(t, lds, lane, wave);
    if constexpr (J < 6 + log2i(NW))
        group_rounds<NW, J + 1>(t, lds, lane, wave);
}

// ---------------------------------------------------------------- wave utils

// The value of x, hidden from the optimiser.  Persistent kernels re-derive
// their lane index through this at the top of every tile so that the 64
// per-register address constants computed from it are not hoisted out of the
// tile loop (which would keep them all live in registers).
__device__ __forceinline__ uint32_t opaque(uint32_t x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
template <class T>
__device__ __forceinline__ T *uniform(T *p)
{
    const uint64_t b = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<T *>(((uint64_t)uniform((uint32_t)(b >> 32)) << 32) | uniform((uint32_t)b));
}

// ------------------------------------- sort of u32 keys, mirrored merge rounds
//
// The tile and group sorts of u32 keys.  Every run ascends; a merge of two
// runs starts by comparing position i of the pair with its mirror 2L - 1 - i
// (which leaves the lower half's keys in the first run's place and both
// places bitonic), so no run has to descend and no register is complemented
// for its direction: the mirror is an address (the partner run is read from
// the LDS in reverse) or a lane pattern.  The stages of round J are position
// bits 5+J .. 0; bits 5 .. 0 are registers in BLOCKED layout.
//   Rounds 1..3 bring lane bits 0..2 together by DPP moves inside eight lanes:
//     two VALU instructions per key and stage, and no LDS.  (Each round through
//     the LDS costs two transposes, 512 cycles of the CU's one LDS pipe; the
//     DPP stages of rounds 1..3 together cost 6 x 64 more VALU instructions on
//     one of four SIMDs.)
//   Rounds 4 and 5 use a third layout,
//       SPLIT    register = p bits 6..10 and p bit 5, lane = p bits 0..4 and p bit 11
//     which is what the two 32 x 32 block transposes of the half-width scheme
//     leave without the exchange of quadrants.
//   Round 6 (p bit 11) takes the half-width transposes to STRIDED and back.  The
//     upper half of the tile is complemented from the start of the sort (it
//     ends rounds 1..5 descending), so this round needs no mirror.
// A wave needs 9 KiB of LDS for all of it, and 64 registers of keys plus what
// addresses take: four waves fit per SIMD.

// Lane patterns of a DPP move: the partner lane inside four or eight lanes.
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppXor3 = 0x1B, kDppXor7 = 0x141;

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}

// One stage against the partner lane: `keep` is 0 in the lanes that take the
// smaller key and ~0 in those that take the larger one, so that the median of
// both keys and `keep` is the one to keep.
template <int CTRL>
__device__ __forceinline__ void lane_clean(Lines<false> &t, uint32_t keep)
{
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        t.k[r] = med3(t.k[r], dpp_move<CTRL>(t.k[r]), keep);
}

// The same against the mirrored register of the partner lane.
template <int CTRL>
__device__ __forceinline__ void lane_clean_mirrored(Lines<false> &t, uint32_t keep)
{
#pragma unroll
    for (int r = 0; r < kLine / 2; ++r) {
        const uint32_t a = t.k[r], b = t.k[kLine - 1 - r];
        t.k[r] = med3(a, dpp_move<CTRL>(b), keep);
        t.k[kLine - 1 - r] = med3(b, dpp_move<CTRL>(a), keep);
    }
}

// BLOCKED -> SPLIT.  J > 0: with the partner runs of merge round J mirrored:
// the registers whose bit J - 1 (p bit 5+J) is set take the key of the
// position with bits 0 .. 4+J inverted.
template <int J>
__device__ __forceinline__ void blocked_to_split(uint32_t (&x)[kLine], uint32_t *lds, uint32_t lane)
{
    static_assert(J < 6, "the mirror stays inside a half-wave's block");
    constexpr int H = kLine / 2;
    uint32_t *m = half_matrix(lds, lane);
    const uint32_t l = lane & 31;
    uint32_t *row = static_cast<uint32_t *>(__builtin_assume_aligned(m + kHalfStride * l, 16));
    uint32_t y[kLine];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int c = 0; c < H; ++c)
            row[c] = x[H * h + c];
        wave_lds_fence();
#pragma unroll
        for (int r = 0; r < H; ++r) {
            const bool mirror = J > 0 && ((r >> (J > 0 ? J - 1 : 0)) & 1);
            if (mirror)
                y[H * (1 - h) + r] = m[kHalfStride * (r ^ ((1 << (J > 0 ? J - 1 : 0)) - 1)) + (31 - l)];
            else
                y[H * h + r] = m[kHalfStride * r + l];
        }
        wave_lds_fence();
    }
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        x[r] = y[r];
}

// SPLIT -> BLOCKED.
__device__ __forceinline__ void split_to_blocked(uint32_t (&x)[kLine], uint32_t *lds, uint32_t lane)
{
    half_block_transpose<0, true>(x, lds, lane);
    half_block_transpose<kLine / 2, true>(x, lds, lane);
}

// Sort a wave tile of u32 keys: on entry any order (64 keys per lane), on exit
// sorted in BLOCKED layout.
__device__ __forceinline__ void sort_tile_keys(Lines<false> &t, uint32_t *lds, uint32_t lane)
{
    const uint32_t upper = opaque(0u - (lane >> 5));  // ~0 in the tile's upper half
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        t.k[r] ^= upper;
    oe_sort_lines<0, kLine - 1>(t);
    const uint32_t b0 = opaque(0u - (lane & 1)), b1 = opaque(0u - ((lane >> 1) & 1)), b2 = opaque(0u - ((lane >> 2) & 1));
    lane_clean_mirrored<kDppXor1>(t, b0);
    half_clean_lines<kLine / 2, -1>(t);
    lane_clean_mirrored<kDppXor3>(t, b1);
    lane_clean<kDppXor1>(t, b0);
    half_clean_lines<kLine / 2, -1>(t);
    lane_clean_mirrored<kDppXor7>(t, b2);
    lane_clean<kDppXor2>(t, b1);
    lane_clean<kDppXor1>(t, b0);
    half_clean_lines<kLine / 2, -1>(t);
    blocked_to_split<4>(t.k, lds, lane);
    half_clean_lines<8, -1>(t);
    split_to_blocked(t.k, lds, lane);
    half_clean_lines<kLine / 2, -1>(t);
    blocked_to_split<5>(t.k, lds, lane);
    half_clean_lines<16, -1>(t);
    split_to_blocked(t.k, lds, lane);
    half_clean_lines<kLine / 2, -1>(t);
    to_strided_half(t, lds, lane);
#pragma unroll
    for (int r = kLine / 2; r < kLine; ++r)
        t.k[r] = ~t.k[r];
    half_clean_lines<kLine / 2, -1>(t);
    to_blocked_half(t, lds, lane);
    half_clean_lines<kLine / 2, -1>(t);
}

// The same sort of a wave tile of 64-bit elements, key/value ones or u64 keys: a
// stage between lanes takes two moves, a comparison and two selects per element
// (five VALU instructions against two for a key), which still undercuts the
// two transposes of both 32-bit halves that a round through the LDS costs.
template <int CTRL>
__device__ __forceinline__ uint64_t dpp_move(uint64_t x)
{
    const uint32_t hi = dpp_move<CTRL>((uint32_t)(x >> 32)), lo = dpp_move<CTRL>((uint32_t)x);
    return ((uint64_t)hi << 32) | lo;
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x)
{
    return elem_of(dpp_move<CTRL>(bits_of(x)));
}

// The smaller of x and y, or the larger; equal elements are alike in every bit.
template <class E>
__device__ __forceinline__ E keep_elem(E x, E y, bool larger)
{
    return ((x < y) != larger) ? x : y;
}

template <int CTRL, class E>
__device__ __forceinline__ void lane_clean(E (&x)[kLine], bool larger)
{
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        x[r] = keep_elem(x[r], dpp_move<CTRL>(x[r]), larger);
}

template <int CTRL, class E>
__device__ __forceinline__ void lane_clean_mirrored(E (&x)[kLine], bool larger)
{
#pragma unroll
    for (int r = 0; r < kLine / 2; ++r) {
        const E a = x[r], b = x[kLine - 1 - r];
        x[r] = keep_elem(a, dpp_move<CTRL>(b), larger);
        x[kLine - 1 - r] = keep_elem(b, dpp_move<CTRL>(a), larger);
    }
}

template <int J, class E>
__device__ __forceinline__ void blocked_to_split_wide(E (&x)[kLine], uint32_t *lds, uint32_t lane)
{
    uint32_t hi[kLine], lo[kLine];
    split_halves(x, hi, lo);
    blocked_to_split<J>(hi, lds, lane);
    blocked_to_split<J>(lo, lds, lane);
    join_halves(x, hi, lo);
}

template <class E>
__device__ __forceinline__ void split_to_blocked_wide(E (&x)[kLine], uint32_t *lds, uint32_t lane)
{
    uint32_t hi[kLine], lo[kLine];
    split_halves(x, hi, lo);
    split_to_blocked(hi, lds, lane);
    split_to_blocked(lo, lds, lane);
    join_halves(x, hi, lo);
}

// The element in reversed order (see flip).
__device__ __forceinline__ double complement(double x) { return elem_of(bits_of(x) ^ kPayloadMask); }
__device__ __forceinline__ uint64_t complement(uint64_t x) { return ~x; }

template <class L>
__device__ __forceinline__ void sort_tile_wide(L &t, uint32_t *lds, uint32_t lane)
{
    flip(t, lane >> 5);
    oe_sort_lines<0, kLine - 1>(t);
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
    lane_clean_mirrored<kDppXor1>(t.e, b0);
    half_clean_lines<kLine / 2, -1>(t);
    lane_clean_mirrored<kDppXor3>(t.e, b1);
    lane_clean<kDppXor1>(t.e, b0);
    half_clean_lines<kLine / 2, -1>(t);
    lane_clean_mirrored<kDppXor7>(t.e, b2);
    lane_clean<kDppXor2>(t.e, b1);
    lane_clean<kDppXor1>(t.e, b0);
    half_clean_lines<kLine / 2, -1>(t);
    blocked_to_split_wide<4>(t.e, lds, lane);
    half_clean_lines<8, -1>(t);
    split_to_blocked_wide(t.e, lds, lane);
    half_clean_lines<kLine / 2, -1>(t);
    blocked_to_split_wide<5>(t.e, lds, lane);
    half_clean_lines<16, -1>(t);
    split_to_blocked_wide(t.e, lds, lane);
    half_clean_lines<kLine / 2, -1>(t);
    to_strided_half(t, lds, lane);
#pragma unroll
    for (int r = kLine / 2; r < kLine; ++r)
        t.e[r] = complement(t.e[r]);
    half_clean_lines<kLine / 2, -1>(t);
    to_blocked_half(t, lds, lane);
    half_clean_lines<kLine / 2, -1>(t);
}

// Group sort of u32 keys: 8 waves, sub-tiles of 4096 keys, each sorted in
// BLOCKED layout by its wave; rounds 7..9 merge across the waves through the
// CROSS layout, half of the group's keys at a time, so that the shared LDS is
// the waves' own 9 KiB slices side by side (72 KiB: two groups fit a CU).
// A step stores the keys of one value of a p bit that is a register bit on
// both sides, at word 2304 (p bits 12..14) + 68 (five of p bits 6..11) + p bits
// 0..5: lane-consecutive 4-byte accesses and 16-byte accesses of rows 68 words
// apart, both conflict-free.  In both exchanges a wave writes or reads only its
// own slice on the BLOCKED / SPLIT side, which saves a barrier.
constexpr int kKeyGroupWaves = 8;

// BLOCKED p = 4096 wave + 64 lane + r  ->  CROSS (lane = p bits 0..5, wave = p
// bits 6..8, register = p bits 9..14) for round J = 7..9: the registers whose
// bit J - 4 (p bit 5+J) is set take the key of the position with bits 0..4+J
// inverted.  After the exchange of quadrants p bit 11 is register bit 5 on
// the BLOCKED side and register bit 2 on the CROSS side.
template <int J>
__device__ __forceinline__ void keys_to_cross(uint32_t (&x)[kLine], uint32_t *lds, uint32_t lane, uint32_t wave)
{
    constexpr int H = kLine / 2;
    swap_quadrants(x);
    uint32_t *w = static_cast<uint32_t *>(__builtin_assume_aligned(
        lds + kHalfLdsWords * wave + kLdsStride * (lane & 31) + H * (lane >> 5), 16));
    const uint32_t *same = lds + kLdsStride * wave + lane;
    const uint32_t *mirror = lds + kLdsStride * (kKeyGroupWaves - 1 - wave) + (kWave - 1 - lane);
    uint32_t y[kLine];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int r = 0; r < H; ++r)
            w[r] = x[H * h + r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kLine; ++r) {
            const bool up = (r >> (J - 4)) & 1;
            const int src = up ? r ^ ((1 << (J - 4)) - 1) : r;
            if (((src >> 2) & 1) == h)
                y[r] = (up ? mirror : same)[kHalfLdsWords * (src >> 3) + kLdsStride * 8 * (src & 3)];
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        x[r] = y[r];
}

// CROSS -> SPLIT (p bit 10 is register bit 1 of CROSS and bit 4 of SPLIT).
__device__ __forceinline__ void cross_to_split(uint32_t (&x)[kLine], uint32_t *lds, uint32_t lane, uint32_t wave)
{
    constexpr int H = kLine / 2;
    uint32_t *w = lds + kLdsStride * wave + lane;
    const uint32_t *own = lds + kHalfLdsWords * wave + kLdsStride * 16 * (lane >> 5) + (lane & 31);
    uint32_t y[kLine];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (h)
            __syncthreads();
#pragma unroll
        for (int r = 0; r < kLine; ++r)
            if (((r >> 1) & 1) == h)
                w[kHalfLdsWords * (r >> 3) + kLdsStride * (8 * (r & 1) + 16 * ((r >> 2) & 1))] = x[r];
        __syncthreads();
#pragma unroll
        for (int s = 0; s < kLine; ++s)
            if (((s >> 4) & 1) == h)
                y[s] = own[kLdsStride * (s & 15) + H * (s >> 5)];
    }
    wave_lds_fence();  // the next writes of this slice are the wave's own
#pragma unroll
    for (int r = 0; r < kLine; ++r)
        x[r] = y[r];
}

template <int J>
__device__ __forceinline__ void group_round_keys(Lines<false> &t, uint32_t *lds, uint32_t lane, uint32_t wave)
{
    keys_to_cross<J>(t.k, lds, lane, wave);
    half_clean_lines<(1 << (J - 4)), -1>(t);  // p bits 5+J .. 9
    cross_to_split(t.k, lds, lane, wave);
    half_clean_lines<4, -1>(t);  // p bits 8 .. 6
    split_to_blocked(t.k, lds + kHalfLdsWords * wave, lane);
    half_clean_lines<kLine / 2, -1>(t);
}

// The rounds that a group of `count` keys needs: a run that reaches the last key
// is merged with padding only.
__device__ __forceinline__ void group_rounds_keys(Lines<false> &t, uint32_t *lds, uint32_t lane, uint32_t wave,
                                                  uint32_t count)
{
    if (count > kTile)
        group_round_keys<7>(t, lds, lane, wave);
    if (count > 2 * kTile)
        group_round_keys<8>(t, lds, lane, wave);
    if (count > 4 * kTile)
        group_round_keys<9>(t, lds, lane, wave);
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

// Co-rank (merge-path split) of the stable merge of sorted A and B: the number
// of elements of A among the first d outputs when equal keys take A first.
// It is the smallest i in [max(0, d-nb), min(d, na)] with A[i] > B[d-1-i].
// Lanes 0..31 search for diagonal d of their half-wave, lanes 32..63 for
// theirs; each round probes 32 evenly spaced candidates per half and keeps
// the bracket between the last failing and the first passing probe, so a
// search over 2^25 candidates takes 5 rounds of loads.
template <class K>
__device__ __forceinline__ uint32_t corank_halfwave(const K *__restrict__ A, uint32_t na, const K *__restrict__ B,
                                                    uint32_t nb, uint32_t d, uint32_t lane)
{
    const uint32_t k = lane & 31;
    const uint32_t shift = lane & 32;  // 0 or 32: position of this half in the ballot
    uint32_t lo = d > nb ? d - nb : 0;
    uint32_t hi = d < na ? d : na;
    while (true) {
        const uint32_t span = hi - lo;
        if (ballot(span != 0) == 0)
            break;
        // probe k of this half: lo + floor(span * k / 32) < hi when span > 0
        const uint32_t i = lo + (uint32_t)(((uint64_t)span * k) >> 5);
        bool pass = true;
        if (span != 0)
            pass = A[i] > B[d - 1 - i];
        const uint32_t fails = (uint32_t)(ballot(!pass && span != 0) >> shift);
        const uint32_t c = __popc(fails);  // probes 0..c-1 fail (the predicate is monotone)
        if (span != 0) {
            if (c == 0) {
                hi = lo;
            } else {
                const uint32_t plast = lo + (uint32_t)(((uint64_t)span * (c - 1)) >> 5);
                const uint32_t pnext = c < 32 ? lo + (uint32_t)(((uint64_t)span * c) >> 5) : hi;
                lo = plast + 1;
                hi = pnext;
            }
        }
    }
    return lo;
}

}  // namespace bcf
