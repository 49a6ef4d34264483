// Device planning of table-driven sorts and merges whose run or segment
// offsets live in device memory: the block-sort tile list, and for every
// merge pass its job list and tile-to-job map, are computed by small kernels
// from the offsets, so that nothing is read back to the host and a captured
// graph stays valid when the offsets change between replays (as long as the
// total stays within the capacity the temp buffer was sized for).
//
// The merges are the paper's merging (Sec. 3.2) of groups of runs: group g's
// runs are merged four at a time (or pairwise, when the tuning asks for it), pass
// after pass, until one run remains; every group has its own pass count and
// buffer parity, so its last pass writes the output.  Calls on few keys are
// bound by the launches, whose number only depends on what the host knows (the
// capacity and the number of offsets): four planner launches, then two per
// four-way level, which takes the jobs of two runs and the copies along.
// Three kinds of groups:
//   * merge_runs: one group of k explicit runs [off[r], off[r+1]);
//   * buckets (the final merge after a distribution, Sec. 3.2 and 3.3): group
//     b holds the s pieces [off[b s + r], off[b s + r + 1]) of bucket b; a
//     pivot bucket holds one key value, so its pieces are already merged and
//     the group is one copy;
//   * segments: segment g = [off[g], off[g+1]) is block-sorted into runs of
//     4096 keys (wave tiles) or of a group tile (long segments), then those
//     runs are merged.
// The tables are the same BlockTile / MergeJob / tile-to-job tables the host
// planner of bcf_api.hip builds, read by the same kernels, which take their
// tile counts from device words written here.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstring>
#include <mutex>
#include <thread>
#include <utility>
#include <vector>

#include "bcf.h"
#include "bcf_device.hpp"
#include "bcf_internal.hpp"

namespace bcf {

// Host services of bcf_api.hip: a profiling scope around one launch.
void *prof_begin(const char *name, hipStream_t s, double bytes);
void prof_end(void *scope);

namespace {

#define BCF_PLAN_TRY(x)                     \
    do {                                    \
        bcf_status st_ = (x);               \
        if (st_ != BCF_OK)                  \
            return st_;                     \
    } while (0)

constexpr int kMaxPlanPasses = 24;  // 4096 << 24 keys > 2^32
constexpr int kMaxPlan4Passes = 12; // fan-in 4 steps: 4096 << 24 keys > 2^32
constexpr uint32_t kPlanBlock = 256;
constexpr uint64_t kMaxKeys = 0xFFFFFFFFull;

uint64_t a256(uint64_t x) { return (x + 255) & ~uint64_t(255); }

uint32_t clog2(uint64_t x)
{
    uint32_t p = 0;
    while ((uint64_t(1) << p) < x)
        ++p;
    return p;
}

__host__ __device__ inline uint32_t ceil_log2_u(uint64_t x)
{
    uint32_t p = 0;
    while ((uint64_t(1) << p) < x)
        ++p;
    return p;
}

enum GroupKind : uint32_t { kKindRuns = 0, kKindBuckets = 1, kKindSegments = 2 };

// One group as the planner sees it: `steps4` fan-in 4 steps, or `merges` binary
// ones, until one run remains.
struct GroupInfo {
    uint32_t first;   // explicit runs: index of the group's first offset
    uint32_t nruns;   // runs before the merge passes
    uint32_t steps4;  // fan-in 4 steps
    uint32_t merges;  // binary steps (none under fan-in 4)
    uint32_t passes;  // the steps, one more with a final copy, or 1 copy
    uint32_t run0;    // segments: run length after the block sort (0: explicit runs)
    uint64_t start, end;
};

// Everything the planner kernels read: the offsets, the kind of groups, and
// where the tables go.
struct PlanArgs {
    const uint64_t *off;
    uint32_t kind;
    uint32_t G;          // groups
    uint32_t k;          // explicit runs: offsets k + 1
    uint32_t s;          // buckets: runs (pieces) per bucket
    uint32_t pivot;      // buckets: odd buckets are pivot buckets
    uint32_t extra_copy; // runs: one more pass copying temp into the output
    uint64_t gmin;       // segments: group tiles from this many keys (and more than 4096)
    uint32_t grun;       // segments: keys per group tile
    uint32_t PM;         // merge passes planned
    uint32_t four;       // fan-in 4 steps (PM4 passes, PM = 0) or binary ones (PM passes, PM4 = 0)
    uint32_t PM4;        // at most kMaxPlan4Passes
    uint64_t cap;        // the most keys: what the temp buffer holds, or the arrays where they hold less
    uint64_t *total;     // host word for the last offset, or nullptr
    uint32_t *status;    // 0: plan valid; 1: offsets invalid or past the capacity
    // block-sort tiles (segments): counts per group, prefix, lists, totals
    uint32_t *bw, *bg;
    BlockTile *wtiles, *gtiles;
    uint32_t wb, gb;     // list bounds
    uint32_t *wcount, *gcount;
    // merge pass j (0-based): job counts per group (prefix), jobs, tiles per job (prefix), tile map, total
    uint32_t *gjob[kMaxPlanPasses];
    MergeJob *jobs[kMaxPlanPasses];
    uint32_t *jtile[kMaxPlanPasses];
    uint32_t *tjob[kMaxPlanPasses];
    uint32_t jb[kMaxPlanPasses], tb[kMaxPlanPasses];  // bounds
    uint32_t *tcount;    // [PM] tiles of each pass
    // fan-in 4 pass j: job counts per group (prefix), jobs, per-job searches /
    // item slots / cut records (prefix: the jobs' first indices), and the
    // pass's counts (jobs, searches, item slots); bounds
    uint32_t *gjob4[kMaxPlan4Passes];
    Merge4Job *jobs4[kMaxPlan4Passes];
    uint32_t *jt4[kMaxPlan4Passes], *ji4[kMaxPlan4Passes], *jr4[kMaxPlan4Passes];
    uint32_t *c4[kMaxPlan4Passes];
    uint32_t j4b[kMaxPlan4Passes];
    uint32_t t4b, i4b, r4b;
};
static_assert(sizeof(PlanArgs) <= 4096, "kernel arguments are limited to 4 KiB");

__device__ GroupInfo group_info(const PlanArgs &a, uint32_t g)
{
    GroupInfo gi;
    if (a.kind == kKindSegments) {
        gi.start = a.off[g];
        gi.end = a.off[g + 1];
        const uint64_t len = gi.end - gi.start;
        gi.run0 = (len > (uint64_t)kTile && len >= a.gmin) ? a.grun : (uint32_t)kTile;
        gi.nruns = (uint32_t)((len + gi.run0 - 1) / gi.run0);
        uint32_t r = gi.nruns;
        gi.steps4 = 0;
        while (a.four && r > 1 && gi.steps4 < a.PM4) {
            r = (r + 3) / 4;
            ++gi.steps4;
        }
        gi.merges = a.four ? 0 : ceil_log2_u(r);
        gi.passes = gi.steps4 + gi.merges;
        gi.first = 0;
    } else {
        gi.run0 = 0;
        gi.steps4 = 0;
        if (a.kind == kKindRuns) {
            gi.first = 0;
            gi.nruns = a.k;
        } else {
            gi.first = g * a.s;
            gi.nruns = a.s;
        }
        const bool pivot = a.kind == kKindBuckets && a.pivot && (g & 1u);
        uint32_t r = gi.nruns;
        while (a.four && !pivot && r > 1 && gi.steps4 < a.PM4) {
            r = (r + 3) / 4;
            ++gi.steps4;
        }
        gi.merges = pivot || a.four ? 0 : ceil_log2_u(r);
        const uint32_t levels = gi.steps4 + gi.merges;
        if (a.kind == kKindRuns)
            gi.passes = levels + (a.extra_copy ? 1 : 0);
        else
            gi.passes = levels ? levels : 1;  // a group of one run (or a pivot bucket) is copied
        gi.start = a.off[gi.first];
        gi.end = a.off[gi.first + gi.nruns];
    }
    return gi;
}

// Offset of run boundary r (0 <= r <= nruns) of a group.
__device__ uint64_t run_bound(const PlanArgs &a, const GroupInfo &gi, uint32_t r)
{
    if (gi.run0) {
        const uint64_t p = gi.start + (uint64_t)r * gi.run0;
        return p < gi.end ? p : gi.end;
    }
    return a.off[gi.first + r];
}

// Binary jobs of pass j (1-based).
__device__ uint32_t jobs_in(const GroupInfo &gi, uint32_t j)
{
    if (gi.end == gi.start || j > gi.passes)
        return 0;
    if (j <= gi.merges) {
        const uint64_t span = 1ull << j;
        return (uint32_t)((gi.nruns + span - 1) / span);
    }
    return 1;  // the copy pass
}

// Fan-in 4 jobs of pass j (1-based): groups of four runs of 4^(j-1) run0 keys.
__device__ uint32_t jobs4_in(const GroupInfo &gi, uint32_t j)
{
    if (gi.end == gi.start || j > gi.passes)
        return 0;
    if (j <= gi.steps4) {
        const uint64_t span = 1ull << (2 * j);
        return (uint32_t)((gi.nruns + span - 1) / span);
    }
    return 1;  // the copy pass
}

// Buffer of group gi after its pass j (0: after the block sort, segments);
// its last pass writes the output.
__device__ uint16_t buf_after(const GroupInfo &gi, uint32_t j)
{
    return ((gi.passes - j) % 2 == 0) ? (uint16_t)kBufOut : (uint16_t)kBufTemp;
}

// The words the other planner kernels accumulate into or test start at zero:
// status, block-tile totals, pass totals.
__global__ void k_plan_zero(PlanArgs a)
{
    if (threadIdx.x == 0) {
        *a.status = 0;
        *a.wcount = 0;
        *a.gcount = 0;
    }
    for (uint32_t j = threadIdx.x; j < kMaxPlanPasses; j += blockDim.x)
        a.tcount[j] = 0;
}

// (before the checks: the launch ends when the store has reached the host)
__device__ void report_total(const PlanArgs &a, uint32_t noff)
{
    if (a.total)
        __hip_atomic_store(a.total, a.off[noff - 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Validity of the offsets: off[0] == 0, nondecreasing, total within the
// capacity.  One thread per offset pair; any failure sets the status word.
__global__ __launch_bounds__(kPlanBlock) void k_plan_check(PlanArgs a, uint32_t noff)
{
    const uint32_t i = blockIdx.x * kPlanBlock + threadIdx.x;
    if (i == 0)
        report_total(a, noff);
    if (i == 0 && (a.off[0] != 0 || a.off[noff - 1] > a.cap))
        *a.status = 1;
    if (i + 1 < noff && a.off[i + 1] < a.off[i])
        *a.status = 1;
}

// Both at once, by one work-group, when the offsets are few: a launch less.
// 32768 offsets take it 12 us, the two launches 9.
constexpr uint32_t kScanBlock = 1024;
constexpr uint32_t kBeginMaxOffsets = 1u << 14;

__global__ __launch_bounds__(kScanBlock) void k_plan_begin(PlanArgs a, uint32_t noff)
{
    if (threadIdx.x == 0)
        report_total(a, noff);
    bool bad = false;
#pragma unroll 8
    for (uint32_t i = threadIdx.x; i < noff; i += kScanBlock) {
        const uint64_t x = a.off[i], y = a.off[i + 1 < noff ? i + 1 : i];
        bad |= y < x || (i == 0 && x != 0) || (i == noff - 1 && x > a.cap);
    }
    const int any = __syncthreads_or(bad);
    if (threadIdx.x == 0) {
        *a.status = any ? 1 : 0;
        *a.wcount = 0;
        *a.gcount = 0;
    }
    for (uint32_t j = threadIdx.x; j < kMaxPlanPasses; j += kScanBlock)
        a.tcount[j] = 0;
}

// Exclusive prefix sum of get(0), ..., get(len - 1) into v, v[len] = total
// (also to *total when set), by one work-group in chunks of kScanBlock *
// kScanPer elements: each thread sums kScanPer consecutive elements, the
// waves scan those sums, and each thread writes its elements' prefixes.
// get(i) may read v[i].
constexpr uint32_t kScanPer = 4;

template <class Get>
__device__ void block_scan(uint32_t *v, uint32_t len, uint32_t *total, const Get &get)
{
    __shared__ uint32_t wtot[kScanBlock / kWave];
    const uint32_t lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    uint32_t carry = 0;  // the same in every thread
    for (uint32_t base = 0; base < len; base += kScanBlock * kScanPer) {
        const uint32_t i0 = base + threadIdx.x * kScanPer;
        uint32_t x[kScanPer], sum = 0;
#pragma unroll
        for (uint32_t e = 0; e < kScanPer; ++e) {
            x[e] = i0 + e < len ? get(i0 + e) : 0;
            sum += x[e];
        }
        uint32_t incl = sum;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)incl, d);
            incl += lane >= (uint32_t)d ? y : 0;
        }
        if (lane == kWave - 1)
            wtot[wave] = incl;
        __syncthreads();
        uint32_t before = 0, all = 0;
#pragma unroll
        for (uint32_t w = 0; w < kScanBlock / kWave; ++w) {
            before += w < wave ? wtot[w] : 0;
            all += wtot[w];
        }
        uint32_t run = carry + before + incl - sum;  // prefix of this thread's first element
#pragma unroll
        for (uint32_t e = 0; e < kScanPer; ++e) {
            if (i0 + e < len)
                v[i0 + e] = run;
            run += x[e];
        }
        carry += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        v[len] = carry;
        if (total)
            *total = carry;
    }
}

// Counts per group and their prefix sums, one work-group per array: x = 0 wave
// tiles, 1 group tiles (segments), 2 + j binary jobs of pass j, 2 + PM + j
// fan-in 4 jobs of pass j.
__global__ __launch_bounds__(kScanBlock) void k_plan_groups(PlanArgs a, uint32_t first_array)
{
    const uint32_t x = blockIdx.x + first_array;
    const bool ok = *a.status == 0;
    uint32_t *v = x == 0 ? a.bw : x == 1 ? a.bg : x < 2 + a.PM ? a.gjob[x - 2] : a.gjob4[x - 2 - a.PM];
    uint32_t *total = x == 0 ? a.wcount : x == 1 ? a.gcount : nullptr;
    block_scan(v, a.G, total, [&](uint32_t g) -> uint32_t {
        if (!ok)
            return 0;
        const GroupInfo gi = group_info(a, g);
        if (x < 2)
            return (gi.run0 > (uint32_t)kTile) == (x == 1) ? gi.nruns : 0;
        return x < 2 + a.PM ? jobs_in(gi, x - 1) : jobs4_in(gi, x - 1 - a.PM);
    });
}

// Largest i in [0, n) with v[i] <= x (v nondecreasing, v[0] <= x).
__device__ uint32_t upper_index(const uint32_t *v, uint32_t n, uint32_t x)
{
    uint32_t lo = 0, hi = n;  // v[lo] <= x, answer in [lo, hi)
    while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (v[mid] <= x)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// Block-sort tiles (segments): slot t of the wave or group list.
__device__ void plan_block_tile(const PlanArgs &a, bool group, uint32_t t)
{
    const uint32_t *pre = group ? a.bg : a.bw;
    if (t >= (group ? a.gb : a.wb) || t >= pre[a.G])
        return;
    const uint32_t g = upper_index(pre, a.G, t);
    const GroupInfo gi = group_info(a, g);
    const uint64_t o = (uint64_t)(t - pre[g]) * gi.run0;
    BlockTile b;
    b.start = gi.start + o;
    b.count = (uint32_t)min<uint64_t>(gi.run0, gi.end - gi.start - o);
    b.dst = buf_after(gi, 0);
    (group ? a.gtiles : a.wtiles)[t] = b;
}

// Jobs of every pass: thread (j, slot) builds job `slot` of pass j from its
// group's run boundaries and writes its tile count.
__global__ __launch_bounds__(kPlanBlock) void k_plan_jobs(PlanArgs a)
{
    const uint32_t j = blockIdx.y;  // 0-based pass
    const uint32_t slot = blockIdx.x * kPlanBlock + threadIdx.x;
    const uint32_t *pre = a.gjob[j];
    const uint32_t total = min(pre[a.G], a.jb[j]);
    if (slot >= total)
        return;
    const uint32_t g = upper_index(pre, a.G, slot);
    const uint32_t q = slot - pre[g];
    const GroupInfo gi = group_info(a, g);
    const uint32_t pass = j + 1;
    MergeJob m;
    if (pass <= gi.merges) {
        const uint64_t half = 1ull << j, span = 2 * half;  // runs of run0 keys
        const uint64_t r0 = q * span;
        const uint32_t rm = (uint32_t)min<uint64_t>(r0 + half, gi.nruns);
        const uint32_t r1 = (uint32_t)min<uint64_t>(r0 + span, gi.nruns);
        const uint64_t b0 = run_bound(a, gi, (uint32_t)r0), bm = run_bound(a, gi, rm), b1 = run_bound(a, gi, r1);
        m.a_start = b0;
        m.na = (uint32_t)(bm - b0);
        m.nb = (uint32_t)(b1 - bm);
    } else {  // copy pass: the whole group as one run
        m.a_start = gi.start;
        m.na = (uint32_t)(gi.end - gi.start);
        m.nb = 0;
    }
    m.first_tile = 0;
    m.src = pass == 1 ? (gi.run0 ? buf_after(gi, 0) : (uint16_t)kBufIn) : buf_after(gi, pass - 1);
    m.dst = buf_after(gi, pass);
    a.jobs[j][slot] = m;
    a.jtile[j][slot] = (uint32_t)(((uint64_t)m.na + m.nb + kTile - 1) / kTile);
}

// Tile counts of every pass's jobs -> first tiles (one work-group per pass).
__global__ __launch_bounds__(kScanBlock) void k_plan_scan_jobs(PlanArgs a)
{
    const uint32_t j = blockIdx.x;
    const uint32_t njobs = min(a.gjob[j][a.G], a.jb[j]);
    block_scan(a.jtile[j], njobs, a.tcount + j, [&](uint32_t i) { return a.jtile[j][i]; });
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < njobs; i += kScanBlock)
        a.jobs[j][i].first_tile = a.jtile[j][i];
    if (threadIdx.x == 0 && a.tcount[j] > a.tb[j])
        a.tcount[j] = a.tb[j];  // never more tiles than the launches cover
}

// Tile-to-job maps of every pass.
__global__ __launch_bounds__(kPlanBlock) void k_plan_tile_map(PlanArgs a)
{
    const uint32_t j = blockIdx.y;
    const uint32_t t = blockIdx.x * kPlanBlock + threadIdx.x;
    if (t >= a.tb[j] || t >= a.tcount[j])
        return;
    const uint32_t njobs = min(a.gjob[j][a.G], a.jb[j]);
    a.tjob[j][t] = upper_index(a.jtile[j], njobs, t);
}

// Fan-in 4 job `slot` of pass j (0-based; four runs of 4^j runs each of its
// group, or the whole group to copy) and its counts of cut searches, item
// slots and cut records.
__device__ void plan_job4(const PlanArgs &a, uint32_t j, uint32_t slot)
{
    const uint32_t *pre = a.gjob4[j];
    const uint32_t total = min(pre[a.G], a.j4b[j]);
    if (slot >= total)
        return;
    const uint32_t g = upper_index(pre, a.G, slot);
    const uint32_t q = slot - pre[g];
    const GroupInfo gi = group_info(a, g);
    const uint32_t pass = j + 1;
    const uint64_t unit = 1ull << (2 * j), span = 4 * unit;  // runs of run0 keys
    uint64_t b[5];
    for (int t = 0; t <= 4; ++t)
        b[t] = pass <= gi.steps4 ? run_bound(a, gi, (uint32_t)min<uint64_t>(q * span + t * unit, gi.nruns))
                                 : (t ? gi.end : gi.start);
    Merge4Job m;
    m.start = b[0];
    for (int t = 0; t < 4; ++t)
        m.n[t] = (uint32_t)(b[t + 1] - b[t]);
    m.cut_off = m.item_off = m.task_off = 0;
    // the first pass of explicit runs reads the caller's input
    m.src = pass == 1 ? (gi.run0 ? buf_after(gi, 0) : (uint16_t)kBufIn) : buf_after(gi, pass - 1);
    m.dst = buf_after(gi, pass);
    a.jobs4[j][slot] = m;
    const uint64_t ncd = (uint64_t)m.n[2] + m.n[3];
    const uint32_t J = merge4_ab_segments((uint64_t)m.n[0] + m.n[1], ncd), M = merge4_cd_cuts(ncd);
    a.jt4[j][slot] = merge4_tasks(J, M);
    a.ji4[j][slot] = merge4_items(J, M);
    a.jr4[j][slot] = merge4_records(J, M);
}

// The block-sort tiles (segments: rows 0 and 1 of the grid) and the fan-in 4
// jobs of every pass (the other rows).
__global__ __launch_bounds__(kPlanBlock) void k_plan_tables(PlanArgs a)
{
    const uint32_t t = blockIdx.x * kPlanBlock + threadIdx.x, y = blockIdx.y;
    const uint32_t rows = a.kind == kKindSegments ? 2 : 0;
    if (y < rows)
        plan_block_tile(a, y == 1, t);
    else
        plan_job4(a, y - rows, t);
}

// The fan-in 4 jobs' first search, item slot and cut record of every pass
// (one work-group per pass), and the pass's counts.  Counts past the bounds
// the launches and areas were sized for (never, by the bounds' construction)
// leave the pass with no job: nothing is read or written out of range.
__global__ __launch_bounds__(kScanBlock) void k_plan_scan_jobs4(PlanArgs a)
{
    const uint32_t j = blockIdx.x;
    const uint32_t njobs = min(a.gjob4[j][a.G], a.j4b[j]);
    __shared__ uint32_t tot[3];
    block_scan(a.jt4[j], njobs, &tot[0], [&](uint32_t i) { return a.jt4[j][i]; });
    __syncthreads();
    block_scan(a.ji4[j], njobs, &tot[1], [&](uint32_t i) { return a.ji4[j][i]; });
    __syncthreads();
    block_scan(a.jr4[j], njobs, &tot[2], [&](uint32_t i) { return a.jr4[j][i]; });
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < njobs; i += kScanBlock) {
        a.jobs4[j][i].task_off = a.jt4[j][i];
        a.jobs4[j][i].item_off = a.ji4[j][i];
        a.jobs4[j][i].cut_off = a.jr4[j][i];
    }
    if (threadIdx.x == 0) {
        const bool fits = tot[0] <= a.t4b && tot[1] <= a.i4b && tot[2] <= a.r4b;
        a.c4[j][0] = fits ? njobs : 0;
        a.c4[j][1] = fits ? tot[0] : 0;
        a.c4[j][2] = fits ? tot[1] : 0;
    }
}

// ------------------------------------------------------------- host side

struct PlanSpec {
    uint32_t kind;
    uint32_t G, k, s, pivot, extra_copy;
    uint64_t gmin;
    uint32_t grun;
    bool pairs;
    uint32_t noff;  // offsets read (validity check)
    bool four;  // fan-in 4 steps; segmented plans reserve the areas of both fan-ins
    bool reserve_four;  // explicit runs / buckets: size the areas of both fan-ins (temp queries)
};

// Bounds of a plan for at most cap keys.
struct PlanBounds {
    uint32_t PM;
    uint64_t wb, gb;
    uint64_t jb[kMaxPlanPasses], tb[kMaxPlanPasses];
    // fan-in 4 steps: passes, jobs per pass, and cut searches / item slots /
    // cut records of any one pass
    uint32_t PM4;
    uint64_t j4b[kMaxPlan4Passes];
    uint64_t t4b, i4b, r4b;
};

// Merge levels of a group of `runs` runs, four-way or binary.
uint32_t merge_levels(uint64_t runs, bool four)
{
    uint32_t st = 0;
    for (; runs > 1; runs = four ? (runs + 3) / 4 : (runs + 1) / 2)
        ++st;
    return st;
}

// Fan-in 4 levels that a plan of segments of at most cap keys in all may take:
// a segment has runs of grun keys, or of a tile where it is shorter than gmin.
uint32_t segment_levels(const PlanSpec &sp, uint64_t cap)
{
    const uint64_t tiles = (std::min(cap, sp.gmin) + kTile - 1) / kTile, groups = (cap + sp.grun - 1) / sp.grun;
    return merge_levels(std::max(tiles, groups), true);
}

PlanBounds plan_bounds(const PlanSpec &sp, uint64_t cap)
{
    PlanBounds b{};
    const uint64_t tiles = (cap + kTile - 1) / kTile;
    if (sp.kind == kKindSegments) {
        b.PM = clog2(std::max<uint64_t>(tiles, 1));
        b.wb = tiles + sp.G;
        b.gb = (cap + sp.grun - 1) / sp.grun + sp.G;
        for (uint32_t j = 1; j <= b.PM; ++j)
            b.jb[j - 1] = ((tiles + sp.G) >> j) + 1 + sp.G;
        {
            // segment g has at most ceil(len_g / 4096) runs, so step j (of four
            // runs of 4^(j-1) each) at most (tiles + G) / 4^j + G jobs; a job of
            // t keys takes at most t / kAbStep + 1 searches and item slots, and
            // two more cut records
            b.PM4 = merge_levels(tiles, true);
            for (uint32_t j = 1; j <= b.PM4; ++j)
                b.j4b[j - 1] = ((tiles + sp.G) >> (2 * j)) + sp.G + 1;
            const uint64_t most = b.PM4 ? b.j4b[0] : 0;
            b.t4b = b.i4b = (cap + kAbStep - 1) / kAbStep + most;
            b.r4b = b.i4b + 2 * most;
        }
    } else {
        const uint32_t nr = sp.kind == kKindRuns ? sp.k : sp.s;
        // a query reserves the areas of both fan-ins; the last level of either
        // may be a copy (buckets: of a group of one run)
        const uint32_t levels = merge_levels(nr, false), levels4 = merge_levels(nr, true);
        const uint32_t copy = sp.kind == kKindRuns ? (sp.extra_copy ? 1 : 0) : 0;
        const uint32_t least = sp.kind == kKindRuns ? 0 : 1;
        b.PM = sp.four && !sp.reserve_four ? 0 : std::max(levels + copy, least);
        for (uint32_t j = 1; j <= b.PM; ++j) {
            // every group: at most ceil(nr / 2^j) binary jobs while merging,
            // else one copy
            const uint64_t per = j <= levels ? ((uint64_t)nr + (1ull << j) - 1) >> j : 1;
            b.jb[j - 1] = per * sp.G;
        }
        if ((sp.four || sp.reserve_four) && levels4 + copy <= (uint32_t)kMaxPlan4Passes) {
            // step j: ceil(nr / 4^j) jobs per group (a copy: one), every job of t
            // keys at most t / kAbStep + 1 searches and item slots and two more
            // cut records
            b.PM4 = std::max(levels4 + copy, least);
            for (uint32_t j = 1; j <= b.PM4; ++j)
                b.j4b[j - 1] = (((uint64_t)nr + (1ull << (2 * j)) - 1) >> (2 * j)) * sp.G + 1;
            const uint64_t most = b.PM4 ? b.j4b[0] : 0;
            b.t4b = b.i4b = (cap + kAbStep - 1) / kAbStep + most;
            b.r4b = b.i4b + 2 * most;
        }
    }
    for (uint32_t j = 1; j <= b.PM; ++j)
        b.tb[j - 1] = tiles + b.jb[j - 1];
    return b;
}

// Temp layout: data ping-pong (keys [, values]), split list, status word,
// block-tile counts and lists, then per pass the job counts, jobs, tile
// counts and tile map, then the per-pass tile totals.
struct PlanLayout {
    uint64_t data, splits, status, bw, bg, wtiles, gtiles, wcount, gcount, tcount;
    uint64_t gjob[kMaxPlanPasses], jobs[kMaxPlanPasses], jtile[kMaxPlanPasses], tjob[kMaxPlanPasses];
    // fan-in 4 steps: per pass the job counts, jobs, per-job counts and pass
    // counts; one search map, item map and cut record area all passes share
    uint64_t gjob4[kMaxPlan4Passes], jobs4[kMaxPlan4Passes];
    uint64_t jt4[kMaxPlan4Passes], ji4[kMaxPlan4Passes], jr4[kMaxPlan4Passes], c4;
    uint64_t imap4, cuts4;
    uint64_t total;
};

PlanLayout plan_layout(const PlanSpec &sp, const PlanBounds &b, uint64_t cap)
{
    PlanLayout L{};
    uint64_t o = 0;
    L.data = o;
    o += a256(cap * 4) * (sp.pairs ? 2 : 1);
    uint64_t maxtb = 1;
    for (uint32_t j = 0; j < b.PM; ++j)
        maxtb = std::max(maxtb, b.tb[j]);
    L.splits = o;
    o = a256(o + (maxtb + 1) * 4);
    L.status = o;
    L.wcount = o + 4;
    L.gcount = o + 8;
    o = a256(o + 16);
    L.tcount = o;
    o = a256(o + kMaxPlanPasses * 4);
    L.bw = o;
    o = a256(o + ((uint64_t)sp.G + 1) * 4);
    L.bg = o;
    o = a256(o + ((uint64_t)sp.G + 1) * 4);
    L.wtiles = o;
    o = a256(o + (sp.kind == kKindSegments ? b.wb : 0) * sizeof(BlockTile));
    L.gtiles = o;
    o = a256(o + (sp.kind == kKindSegments ? b.gb : 0) * sizeof(BlockTile));
    for (uint32_t j = 0; j < b.PM; ++j) {
        L.gjob[j] = o;
        o = a256(o + ((uint64_t)sp.G + 1) * 4);
        L.jobs[j] = o;
        o = a256(o + b.jb[j] * sizeof(MergeJob));
        L.jtile[j] = o;
        o = a256(o + (b.jb[j] + 1) * 4);
        L.tjob[j] = o;
        o = a256(o + b.tb[j] * 4);
    }
    if (b.PM4) {
        for (uint32_t j = 0; j < b.PM4; ++j) {
            L.gjob4[j] = o;
            o = a256(o + ((uint64_t)sp.G + 1) * 4);
            L.jobs4[j] = o;
            o = a256(o + b.j4b[j] * sizeof(Merge4Job));
            L.jt4[j] = o;
            o = a256(o + (b.j4b[j] + 1) * 4);
            L.ji4[j] = o;
            o = a256(o + (b.j4b[j] + 1) * 4);
            L.jr4[j] = o;
            o = a256(o + (b.j4b[j] + 1) * 4);
        }
        L.c4 = o;
        o = a256(o + kMaxPlan4Passes * 4 * 4);
        L.imap4 = o;
        o = a256(o + b.i4b * 4);
        L.cuts4 = o;
        o = a256(o + b.r4b * 16);
    }
    L.total = o;
    return L;
}

uint64_t plan_need(const PlanSpec &sp, uint64_t cap) { return plan_layout(sp, plan_bounds(sp, cap), cap).total; }

// The most keys a temp buffer of `bytes` holds for this plan (0 if none).
uint64_t plan_capacity(const PlanSpec &sp, uint64_t bytes)
{
    if (plan_need(sp, 0) > bytes)
        return 0;
    uint64_t lo = 0, hi = kMaxKeys;  // need(lo) <= bytes
    while (lo < hi) {
        const uint64_t mid = lo + (hi - lo + 1) / 2;
        if (plan_need(sp, mid) <= bytes)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

bcf_status dev(hipError_t e) { return e == hipSuccess ? BCF_OK : BCF_ERR_DEVICE; }

// Words of pinned host memory that a planner launch writes the last offset to.
// A call holds one until it has been written; kTotalSlots are kept, which calls
// in flight on more threads than that go beyond.
constexpr int kTotalSlots = 16;
std::mutex g_total_mu;
uint64_t *g_total[kTotalSlots];

// The last offset of a call, which the host waits for after its launches: the
// planner's first launch writes it, so that the rest of the call runs on behind
// the wait.  The host reads the word itself: with an event recorded behind the
// launch and waited for, calls of 20 segments of up to 600 keys took 36 us each
// (29 without a report, 28 to 30 so).  The wait lets the host run one call ahead
// of the device, which costs calls that take both the same time up to 5 us (4000
// segments of up to 700 keys 70 -> 74 us).  Not reported in a stream capture (and
// without `out`).
class TotalReport {
public:
    TotalReport(uint64_t *out, hipStream_t s) : out_(out), s_(s)
    {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (!out || hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) {
            out_ = nullptr;
            return;
        }
        {
            const std::lock_guard<std::mutex> hold(g_total_mu);
            for (uint64_t *&w : g_total)
                if (w && !word_)
                    std::swap(w, word_);
        }
        if (!word_) {
            // an allocation must not end the captures of other streams
            hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
            (void)hipThreadExchangeStreamCaptureMode(&mode);
            void *w = nullptr;
            if (hipHostMalloc(&w, sizeof(uint64_t), hipHostMallocCoherent | hipHostMallocPortable) == hipSuccess)
                word_ = static_cast<uint64_t *>(w);
            (void)hipThreadExchangeStreamCaptureMode(&mode);
        }
        if (word_)
            __atomic_store_n(word_, kUnwritten, __ATOMIC_RELAXED);
    }
    TotalReport(const TotalReport &) = delete;
    TotalReport &operator=(const TotalReport &) = delete;
    ~TotalReport()
    {
        if (launched_)
            (void)read();  // a word still to be written is not given back
        if (!word_)
            return;
        {
            const std::lock_guard<std::mutex> hold(g_total_mu);
            for (uint64_t *&w : g_total)
                if (!w && word_)
                    std::swap(w, word_);
        }
        if (word_)
            (void)hipHostFree(word_);
    }
    uint64_t *word() const { return word_; }
    bool failed() const { return out_ && !word_; }
    void launched() { launched_ = word_ != nullptr; }
    // After the call's launches: the total, refused when no call takes it.
    bcf_status wait()
    {
        if (!out_)
            return BCF_OK;
        launched_ = false;
        if (!read())
            return BCF_ERR_DEVICE;
        return *out_ > kMaxKeys ? BCF_ERR_INVALID : BCF_OK;
    }

private:
    // No total that a call takes: offsets that do end so are told by the stream
    // being done with the word as it is.
    static constexpr uint64_t kUnwritten = ~0ull;
    bool read()
    {
        using clock = std::chrono::steady_clock;
        auto ask = clock::now() + std::chrono::microseconds(200);
        hipError_t e = hipErrorNotReady;
        while ((*out_ = __atomic_load_n(word_, __ATOMIC_ACQUIRE)) == kUnwritten) {
            if (e == hipSuccess)
                return true;  // the stream is done
            if (e != hipErrorNotReady) {
                word_ = nullptr;  // it has failed: the word may still be written, and is left to it
                return false;
            }
            if (clock::now() < ask)
                continue;
            e = hipStreamQuery(s_);
            if (e == hipErrorNotReady)
                (void)hipGetLastError();  // no error of a launch
            std::this_thread::yield();
            ask = clock::now() + std::chrono::microseconds(200);
        }
        return true;
    }
    uint64_t *out_, *word_ = nullptr;
    hipStream_t s_;
    bool launched_ = false;
};

// Enqueue the planner kernels and the sort / merge kernels of a plan.  keys
// (and values) in kb / vb; temp holds the layout for capacity cap, the arrays
// `limit` keys: offsets that end past either are invalid.  `total` (or NULL)
// takes the last offset.
bcf_status plan_and_run(const PlanSpec &sp, const uint64_t *off_dev, Bufs kb, Bufs vb, char *temp, uint64_t cap,
                        uint64_t limit, uint64_t *total, hipStream_t s)
{
    const PlanBounds b = plan_bounds(sp, cap);
    const PlanLayout L = plan_layout(sp, b, cap);
    if (b.PM > kMaxPlanPasses || sp.G == 0)
        return BCF_ERR_INVALID;
    const bool segs = sp.kind == kKindSegments;
    // the passes to launch, of one fan-in
    const uint32_t PM = sp.four ? 0 : b.PM, P4 = !sp.four ? 0 : segs ? segment_levels(sp, cap) : b.PM4;
    for (uint32_t j = 0; j < PM; ++j)
        if (b.jb[j] > 0xFFFFFFFFull || b.tb[j] > 0xFFFFFFFFull)
            return BCF_ERR_INVALID;
    if (P4 > b.PM4 || P4 > kMaxPlan4Passes || b.t4b > 0xFFFFFFFFull || b.r4b > 0xFFFFFFFFull)
        return BCF_ERR_INVALID;
    PlanArgs a{};
    a.off = off_dev;
    a.kind = sp.kind;
    a.G = sp.G;
    a.k = sp.k;
    a.s = sp.s;
    a.pivot = sp.pivot;
    a.extra_copy = sp.extra_copy;
    a.gmin = sp.gmin;
    a.grun = sp.grun;
    a.PM = PM;
    a.four = sp.four ? 1 : 0;
    a.PM4 = P4;
    a.cap = std::min(cap, limit);
    TotalReport report(total, s);
    if (report.failed())
        return BCF_ERR_NOMEM;
    a.total = report.word();
    a.status = reinterpret_cast<uint32_t *>(temp + L.status);
    a.bw = reinterpret_cast<uint32_t *>(temp + L.bw);
    a.bg = reinterpret_cast<uint32_t *>(temp + L.bg);
    a.wtiles = reinterpret_cast<BlockTile *>(temp + L.wtiles);
    a.gtiles = reinterpret_cast<BlockTile *>(temp + L.gtiles);
    a.wb = (uint32_t)std::min<uint64_t>(b.wb, 0xFFFFFFFFull);
    a.gb = (uint32_t)std::min<uint64_t>(b.gb, 0xFFFFFFFFull);
    a.wcount = reinterpret_cast<uint32_t *>(temp + L.wcount);
    a.gcount = reinterpret_cast<uint32_t *>(temp + L.gcount);
    a.tcount = reinterpret_cast<uint32_t *>(temp + L.tcount);
    for (uint32_t j = 0; j < PM; ++j) {
        a.gjob[j] = reinterpret_cast<uint32_t *>(temp + L.gjob[j]);
        a.jobs[j] = reinterpret_cast<MergeJob *>(temp + L.jobs[j]);
        a.jtile[j] = reinterpret_cast<uint32_t *>(temp + L.jtile[j]);
        a.tjob[j] = reinterpret_cast<uint32_t *>(temp + L.tjob[j]);
        a.jb[j] = (uint32_t)b.jb[j];
        a.tb[j] = (uint32_t)b.tb[j];
    }
    for (uint32_t j = 0; j < P4; ++j) {
        a.gjob4[j] = reinterpret_cast<uint32_t *>(temp + L.gjob4[j]);
        a.jobs4[j] = reinterpret_cast<Merge4Job *>(temp + L.jobs4[j]);
        a.jt4[j] = reinterpret_cast<uint32_t *>(temp + L.jt4[j]);
        a.ji4[j] = reinterpret_cast<uint32_t *>(temp + L.ji4[j]);
        a.jr4[j] = reinterpret_cast<uint32_t *>(temp + L.jr4[j]);
        a.c4[j] = reinterpret_cast<uint32_t *>(temp + L.c4) + 4 * j;
        a.j4b[j] = (uint32_t)b.j4b[j];
    }
    a.t4b = (uint32_t)b.t4b;
    a.i4b = (uint32_t)b.i4b;
    a.r4b = (uint32_t)b.r4b;
    // status, the block-tile totals and the pass totals start at zero (small fill
    // kernels rather than a memset: the sequence may be captured in a graph)
    if (sp.noff <= kBeginMaxOffsets) {
        hipLaunchKernelGGL(k_plan_begin, dim3(1), dim3(kScanBlock), 0, s, a, sp.noff);
        BCF_PLAN_TRY(dev(hipGetLastError()));
    } else {
        hipLaunchKernelGGL(k_plan_zero, dim3(1), dim3(64), 0, s, a);
        BCF_PLAN_TRY(dev(hipGetLastError()));
        const uint32_t blocks = (sp.noff + kPlanBlock - 1) / kPlanBlock;
        hipLaunchKernelGGL(k_plan_check, dim3(blocks), dim3(kPlanBlock), 0, s, a, sp.noff);
        BCF_PLAN_TRY(dev(hipGetLastError()));
    }
    report.launched();
    const uint32_t arrays = 2 + PM + P4, first = segs ? 0 : 2;
    if (arrays > first) {  // nothing to count when no pass is planned (a lone run merged in place)
        hipLaunchKernelGGL(k_plan_groups, dim3(arrays - first), dim3(kScanBlock), 0, s, a, first);
        BCF_PLAN_TRY(dev(hipGetLastError()));
    }
    if (segs || P4) {
        const uint64_t most = std::max(segs ? std::max(b.wb, b.gb) : 1, P4 ? b.j4b[0] : 1);
        hipLaunchKernelGGL(k_plan_tables, dim3((uint32_t)((most + kPlanBlock - 1) / kPlanBlock), (segs ? 2 : 0) + P4),
                           dim3(kPlanBlock), 0, s, a);
        BCF_PLAN_TRY(dev(hipGetLastError()));
    }
    if (PM) {
        uint64_t mj = 1, mt = 1;
        for (uint32_t j = 0; j < PM; ++j) {
            mj = std::max(mj, b.jb[j]);
            mt = std::max(mt, b.tb[j]);
        }
        hipLaunchKernelGGL(k_plan_jobs, dim3((uint32_t)((mj + kPlanBlock - 1) / kPlanBlock), PM), dim3(kPlanBlock), 0, s,
                           a);
        BCF_PLAN_TRY(dev(hipGetLastError()));
        hipLaunchKernelGGL(k_plan_scan_jobs, dim3(PM), dim3(kScanBlock), 0, s, a);
        BCF_PLAN_TRY(dev(hipGetLastError()));
        hipLaunchKernelGGL(k_plan_tile_map, dim3((uint32_t)((mt + kPlanBlock - 1) / kPlanBlock), PM), dim3(kPlanBlock), 0,
                           s, a);
        BCF_PLAN_TRY(dev(hipGetLastError()));
    }
    if (P4) {
        hipLaunchKernelGGL(k_plan_scan_jobs4, dim3(P4), dim3(kScanBlock), 0, s, a);
        BCF_PLAN_TRY(dev(hipGetLastError()));
    }
    const bool pairs = sp.pairs;
    if (segs) {
        {
            void *p = prof_begin(kname_block_sort(pairs, true), s, 0.0);
            const hipError_t e = launch_block_sort_table(pairs, kb, vb, a.wtiles, a.wb, s, a.wcount);
            prof_end(p);
            BCF_PLAN_TRY(dev(e));
        }
        {
            void *p = prof_begin(kname_block_sort(pairs, true), s, 0.0);
            const hipError_t e = launch_block_sort_group_table(pairs, kb, vb, a.gtiles, a.gb, s, a.gcount);
            prof_end(p);
            BCF_PLAN_TRY(dev(e));
        }
    }
    uint32_t *splits = reinterpret_cast<uint32_t *>(temp + L.splits);
    uint32_t *imap4 = reinterpret_cast<uint32_t *>(temp + L.imap4);
    for (uint32_t j = 0; j < P4; ++j)
        for (int phase = 0; phase < 2; ++phase) {
            static const char *const names[2][2] = {{"cuts4_keys_table", "merge4_keys_table"},
                                                    {"cuts4_pairs_table", "merge4_pairs_table"}};
            void *p = prof_begin(names[pairs][phase], s, 0.0);
            const hipError_t e = launch_merge4_table(kb, a.jobs4[j], a.j4b[j], a.t4b, imap4, a.i4b, temp + L.cuts4, cap,
                                                     phase == 1, s, a.c4[j], vb);
            prof_end(p);
            BCF_PLAN_TRY(dev(e));
        }
    for (uint32_t j = 0; j < PM; ++j)
        for (int phase = 0; phase < 2; ++phase) {
            const bool part = phase == 0;
            void *p = prof_begin(part ? kname_partition(pairs, true) : kname_merge(pairs, true), s, 0.0);
            const hipError_t e = launch_merge_table(pairs, kb, vb, a.jobs[j], a.tjob[j], a.tb[j], splits, part, s,
                                                    a.tcount + j);
            prof_end(p);
            BCF_PLAN_TRY(dev(e));
        }
    return report.wait();
}

// The total of a device offset array (its last entry), read on the host:
// for temp queries only (synchronises the stream).
bcf_status read_total(const uint64_t *off_dev, uint64_t last, hipStream_t s, uint64_t &n)
{
    n = 0;
    if (hipMemcpyAsync(&n, off_dev + last, sizeof(uint64_t), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return BCF_ERR_DEVICE;
    return n > kMaxKeys ? BCF_ERR_INVALID : BCF_OK;
}

// Layout of the keys [and values] ping-pong at the start of a plan's temp.
Bufs key_bufs(const uint32_t *in, uint32_t *out, char *temp) { return Bufs{in, out, reinterpret_cast<uint32_t *>(temp)}; }
Bufs val_bufs(const uint32_t *in, uint32_t *out, char *temp, uint64_t cap)
{
    return Bufs{in, out, reinterpret_cast<uint32_t *>(temp + a256(cap * 4))};
}

// A planned call: query (temp == NULL: the total is read from the device) or
// run with the capacity the temp buffer holds, on arrays of `limit` keys.  The
// capacity alone does not keep a call inside its arrays: it is what the plan
// at hand can do with the buffer, above the keys the buffer was sized for
// (sizes are rounded up, and those of merges reserve what either fan-in and an
// extra copy pass need: 16,000,003 keys in 60 runs, capacity 16,033,536).
bcf_status planned_call(const PlanSpec &worst, const PlanSpec &actual, const uint64_t *off_dev, const uint32_t *kin,
                        const uint32_t *vin, uint32_t *kout, uint32_t *vout, uint64_t limit, uint64_t *total,
                        void *temp, uint64_t *temp_bytes, hipStream_t s)
{
    if (!temp) {
        uint64_t n = 0;
        BCF_PLAN_TRY(read_total(off_dev, worst.noff - 1, s, n));
        *temp_bytes = plan_need(worst, n);
        return BCF_OK;
    }
    if (!kin || !kout || (actual.pairs && (!vin || !vout)))
        return BCF_ERR_INVALID;
    // planned for the arrays where the buffer holds that much (no search over the
    // sizes it could hold, on every call)
    const bool whole = limit <= kMaxKeys && plan_need(actual, limit) <= *temp_bytes;
    const uint64_t cap = whole ? limit : plan_capacity(actual, *temp_bytes);
    if (!whole && plan_need(actual, cap) > *temp_bytes)
        return BCF_ERR_TEMP_TOO_SMALL;
    char *tb = static_cast<char *>(temp);
    const Bufs kb = key_bufs(kin, kout, tb);
    const Bufs vb = actual.pairs ? val_bufs(vin, vout, tb, cap) : Bufs{nullptr, nullptr, nullptr};
    return plan_and_run(actual, off_dev, kb, vb, tb, cap, limit, total, s);
}

uint64_t seg_group_min(bool pairs, uint64_t knob) { return knob ? knob : group_run_keys(pairs) / 2; }

// Fan-in 4 steps unless the tuning asks for binary ones; for explicit runs
// never for more runs than kMaxPlan4Passes steps (a copy among them) reduce.
bool segs_four_way() { return tuning().merge_fan_in != 2; }
bool runs_four_way(uint32_t nr)
{
    return tuning().merge_fan_in != 2 && merge_levels(nr, true) + 1 <= (uint32_t)kMaxPlan4Passes;
}

PlanSpec segments_spec(bool pairs, uint32_t nseg)
{
    PlanSpec sp{};
    sp.kind = kKindSegments;
    sp.G = nseg;
    sp.gmin = seg_group_min(pairs, tuning().group_min_keys);
    sp.grun = group_run_keys(pairs);
    sp.pairs = pairs;
    sp.noff = nseg + 1;
    sp.four = segs_four_way();
    return sp;
}

bcf_status segmented_device(bool pairs, const uint32_t *kin, const uint32_t *vin, uint32_t *kout, uint32_t *vout,
                            const uint64_t *off, uint32_t nseg, uint64_t limit, uint64_t *total, void *temp,
                            uint64_t *temp_bytes, hipStream_t s)
{
    if (!temp_bytes)
        return BCF_ERR_INVALID;
    if (nseg == 0) {
        if (!temp)
            *temp_bytes = 0;
        return BCF_OK;
    }
    if (!off)
        return BCF_ERR_INVALID;
    const PlanSpec sp = segments_spec(pairs, nseg);
    return planned_call(sp, sp, off, kin, vin, kout, vout, limit, total, temp, temp_bytes, s);
}

PlanSpec runs_spec(bool pairs, uint32_t k)
{
    PlanSpec sp{};
    sp.kind = kKindRuns;
    sp.G = 1;
    sp.k = k;
    sp.pairs = pairs;
    sp.noff = k + 1;
    sp.four = runs_four_way(k);
    return sp;
}

// The plan that a temp size is reserved for: it depends neither on whether the
// call is in place nor on the fan-in.
PlanSpec reserved(PlanSpec sp)
{
    sp.extra_copy = 1;
    sp.four = false;
    sp.reserve_four = true;
    return sp;
}

bcf_status merge_runs_device(const uint32_t *keys_in, const uint32_t *vals_in, const uint64_t *run_offsets, uint32_t k,
                             uint32_t *keys_out, uint32_t *vals_out, uint64_t limit, uint64_t *total, void *temp,
                             uint64_t *temp_bytes, hipStream_t s)
{
    if (!temp_bytes)
        return BCF_ERR_INVALID;
    if (k == 0) {
        if (!temp)
            *temp_bytes = 0;
        return BCF_OK;
    }
    if (!run_offsets || k == 0xFFFFFFFFu)
        return BCF_ERR_INVALID;
    const bool pairs = vals_in != nullptr;
    PlanSpec sp = runs_spec(pairs, k);
    const uint32_t merges = merge_levels(k, sp.four);
    const PlanSpec worst = reserved(sp);
    const bool inplace = keys_in == keys_out || (pairs && vals_in == vals_out);
    // in place, a run count whose merge levels are odd would make the first pass
    // read and write the output: one more pass copies the result from temp; a
    // lone run not in place is one copy
    sp.extra_copy = merges == 0 ? (inplace ? 0u : 1u) : ((inplace && merges % 2 == 1) ? 1u : 0u);
    if (temp && tuning().check_runs && keys_in) {
        // sortedness of every run, flagged in a spare word of the plan's
        // status area (synchronises the stream)
        uint64_t n = 0;
        BCF_PLAN_TRY(read_total(run_offsets, k, s, n));
        const uint64_t cap = plan_capacity(sp, *temp_bytes);
        if (plan_need(sp, cap) > *temp_bytes || n > cap)
            return BCF_ERR_TEMP_TOO_SMALL;
        if (n > limit)
            return total ? (*total = n, BCF_OK) : BCF_OK;  // as the device check finds it: nothing is written
        const PlanLayout L = plan_layout(sp, plan_bounds(sp, cap), cap);
        uint32_t *flag_d = reinterpret_cast<uint32_t *>(static_cast<char *>(temp) + L.status + 12);
        uint32_t flag = 0;
        const bool ok = hipMemsetAsync(flag_d, 0, sizeof(uint32_t), s) == hipSuccess &&
                        launch_check_runs(keys_in, run_offsets, k, n, flag_d, s) == hipSuccess &&
                        hipMemcpyAsync(&flag, flag_d, sizeof(uint32_t), hipMemcpyDeviceToHost, s) == hipSuccess &&
                        hipStreamSynchronize(s) == hipSuccess;
        if (!ok)
            return BCF_ERR_DEVICE;
        if (flag)
            return BCF_ERR_UNSORTED_RUN;
    }
    return planned_call(worst, sp, run_offsets, keys_in, vals_in, keys_out, vals_out, limit, total, temp,
                        temp_bytes, s);
}

}  // namespace

}  // namespace bcf

using namespace bcf;

extern "C" {

bcf_status bcf_merge_runs(const uint32_t *keys_in, const uint32_t *vals_in, const uint64_t *run_offsets, uint32_t k,
                          uint32_t *keys_out, uint32_t *vals_out, void *temp, uint64_t *temp_bytes, void *stream)
{
    return merge_runs_device(keys_in, vals_in, run_offsets, k, keys_out, vals_out, kMaxKeys, nullptr, temp,
                             temp_bytes, static_cast<hipStream_t>(stream));
}

bcf_status bcf_merge_runs_within(const uint32_t *keys_in, const uint32_t *vals_in, const uint64_t *run_offsets,
                                 uint32_t k, uint64_t n, uint32_t *keys_out, uint32_t *vals_out, uint64_t *total,
                                 void *temp, uint64_t *temp_bytes, void *stream)
{
    if (!temp)
        return BCF_ERR_INVALID;
    return merge_runs_device(keys_in, vals_in, run_offsets, k, keys_out, vals_out, n, total, temp, temp_bytes,
                             static_cast<hipStream_t>(stream));
}

bcf_status bcf_merge_runs_temp(uint64_t n, uint32_t k, int pairs, uint64_t *temp_bytes)
{
    if (!temp_bytes || n > kMaxKeys || k == 0xFFFFFFFFu)
        return BCF_ERR_INVALID;
    *temp_bytes = k ? plan_need(reserved(runs_spec(pairs != 0, k)), n) : 0;
    return BCF_OK;
}

bcf_status bcf_segmented_sort_temp(uint64_t n, uint32_t nseg, int pairs, uint64_t *temp_bytes)
{
    if (!temp_bytes || n > kMaxKeys)
        return BCF_ERR_INVALID;
    *temp_bytes = nseg ? plan_need(segments_spec(pairs != 0, nseg), n) : 0;
    return BCF_OK;
}

bcf_status bcf_segmented_sort(const uint32_t *keys_in, uint32_t *keys_out, const uint64_t *seg_offsets, uint32_t nseg,
                              void *temp, uint64_t *temp_bytes, void *stream)
{
    return segmented_device(false, keys_in, nullptr, keys_out, nullptr, seg_offsets, nseg, kMaxKeys, nullptr, temp,
                            temp_bytes, static_cast<hipStream_t>(stream));
}

bcf_status bcf_segmented_sort_pairs(const uint32_t *keys_in, const uint32_t *vals_in, uint32_t *keys_out,
                                    uint32_t *vals_out, const uint64_t *seg_offsets, uint32_t nseg, void *temp,
                                    uint64_t *temp_bytes, void *stream)
{
    return segmented_device(true, keys_in, vals_in, keys_out, vals_out, seg_offsets, nseg, kMaxKeys, nullptr, temp,
                            temp_bytes, static_cast<hipStream_t>(stream));
}

bcf_status bcf_segmented_sort_within(const uint32_t *keys_in, const uint32_t *vals_in, uint32_t *keys_out,
                                     uint32_t *vals_out, const uint64_t *seg_offsets, uint32_t nseg, uint64_t n,
                                     int pairs, uint64_t *total, void *temp, uint64_t *temp_bytes, void *stream)
{
    if (!temp)
        return BCF_ERR_INVALID;
    return segmented_device(pairs != 0, keys_in, vals_in, keys_out, vals_out, seg_offsets, nseg, n, total, temp,
                            temp_bytes, static_cast<hipStream_t>(stream));
}

bcf_status bcf_sort_u32_pb(const uint32_t *keys_in, uint32_t *keys_out, uint64_t n, uint32_t P, uint32_t run_keys,
                           int pivot_buckets, void *temp, uint64_t *temp_bytes, void *stream)
{
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (!temp_bytes || n > kMaxKeys || P < 1 || P > 65536 || run_keys < 1)
        return BCF_ERR_INVALID;
    if (n == 0) {
        if (!temp)
            *temp_bytes = 0;
        return BCF_OK;
    }
    const uint64_t s64 = (n + run_keys - 1) / run_keys;
    const uint32_t nb = pivot_buckets ? 2 * P - 1 : P;
    // the distribution step's limits (bcf_distribute_runs)
    if (s64 > (1u << 22) || s64 * P > (1ull << 26) || (uint64_t)nb * s64 > (1ull << 24))
        return BCF_ERR_INVALID;
    const uint32_t s = (uint32_t)s64;
    std::vector<uint64_t> seg(s + 1);
    for (uint32_t r = 0; r <= s; ++r)
        seg[r] = std::min<uint64_t>((uint64_t)r * run_keys, n);
    // temp: the distributed keys, the piece offsets, then one scratch area the
    // three steps use in turn (run sort, distribution, bucket merge)
    uint64_t need_runs = 0, need_dist = 0;
    BCF_PLAN_TRY(bcf_segmented_sort_host(nullptr, nullptr, seg.data(), s, nullptr, &need_runs, st));
    BCF_PLAN_TRY(bcf_distribute_runs(nullptr, seg.data(), s, P, P, pivot_buckets, nullptr, nullptr, nullptr, nullptr,
                                     &need_dist, st));
    PlanSpec sp{};
    sp.kind = kKindBuckets;
    sp.G = nb;
    sp.s = s;
    sp.pivot = pivot_buckets ? 1 : 0;
    sp.noff = nb * s + 1;
    sp.four = runs_four_way(s);
    const uint64_t need_merge = plan_need(reserved(sp), n);  // whatever the fan-in
    const uint64_t d_bytes = a256(n * 4), p_bytes = a256(((uint64_t)nb * s + 1) * 8);
    const uint64_t scratch = std::max(need_runs, std::max(need_dist, need_merge));
    const uint64_t need = d_bytes + p_bytes + scratch;
    if (!temp) {
        *temp_bytes = need;
        return BCF_OK;
    }
    if (!keys_in || !keys_out || keys_in == keys_out)
        return BCF_ERR_INVALID;
    if (*temp_bytes < need)
        return BCF_ERR_TEMP_TOO_SMALL;
    char *tb = static_cast<char *>(temp);
    uint32_t *dist = reinterpret_cast<uint32_t *>(tb);
    uint64_t *pieces = reinterpret_cast<uint64_t *>(tb + d_bytes);
    void *scr = tb + d_bytes + p_bytes;
    uint64_t sb = scratch;
    // sorted runs of run_keys keys into the output, then the distribution of
    // the runs into bucket-major pieces, then every bucket merged into the
    // output (piece offsets stay on the device)
    BCF_PLAN_TRY(bcf_segmented_sort_host(keys_in, keys_out, seg.data(), s, scr, &sb, st));
    sb = scratch;
    BCF_PLAN_TRY(bcf_distribute_runs(keys_out, seg.data(), s, P, P, pivot_buckets, dist, pieces, nullptr, scr, &sb,
                                     st));
    return plan_and_run(sp, pieces, key_bufs(dist, keys_out, static_cast<char *>(scr)), Bufs{nullptr, nullptr, nullptr},
                        static_cast<char *>(scr), n, n, nullptr, st);
}

}  // extern "C"
