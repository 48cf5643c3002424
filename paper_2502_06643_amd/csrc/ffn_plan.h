// Tile plan of the grouped expert FFN, built on the device from expert_counts
// so that no bucket size ever travels to the host.
//
// The plan lists the experts resident on local_gpu that received at least one
// route (or, on the receiving side of the all-to-all, the (source GPU, expert)
// segments of the receive buffer, each naming the expert whose weights it
// uses), largest bucket first (ties: lower expert id), with sanitised bucket
// bounds and, for up to two row-tile heights, the exclusive prefix of their
// row-tile counts.  A GEMM workgroup turns a global row-tile index into
// (expert, first row, row count) by scanning that prefix.
#pragma once
#include <type_traits>
#include "common.h"
#include "ffn_split.h"

namespace moe {

constexpr int kPlanHeader = 16;
constexpr int kPlanExpert = kPlanHeader;                       // [256] expert id
constexpr int kPlanStart = kPlanExpert + MOE_MAX_EXPERTS;      // [256] first row
constexpr int kPlanCount = kPlanStart + MOE_MAX_EXPERTS;       // [256] rows
constexpr int kPlanTiles0 = kPlanCount + MOE_MAX_EXPERTS;      // [257] prefix for tile height bm0
constexpr int kPlanTiles1 = kPlanTiles0 + MOE_MAX_EXPERTS + 4; // [257] prefix for tile height bm1
constexpr int kPlanSegOff = kPlanTiles1 + MOE_MAX_EXPERTS + 4; // [257] see kPlanMerged
constexpr int kPlanSegDelta = kPlanSegOff + MOE_MAX_EXPERTS + 4; // [256]
constexpr int kPlanInts = kPlanSegDelta + MOE_MAX_EXPERTS;
static_assert(kPlanInts * sizeof(int32_t) <= kPlanBytes, "plan area too small");
// header: [0] number of listed experts, [1] total row tiles (bm0), [2] total row tiles (bm1),
//         [3] which of the two tile heights the bf16 GEMMs use: 0 = bm0, 1 = bm1 (see `choice`),
//         [4] 1 + how many row tiles of height bm1 hold at most kSmallTileRows rows
//         [5], [6] k parts of the larger and of the small row tiles when the down projection runs in one round and is
//             cut by cost (RoundSplit in ffn_tiles.h); [5] = 0: it is not
//         [7] 1: the segments of one expert are merged into one bucket
//         [8], [9] tokens whose rows for other GPUs the up and the down projection copy (the first tokens, those after
//             them), [10], [11] this GPU's range of the sorted rows (only in a layer call that may have such rows; the first two
//             are written by the row copy: ffn_late.h)
constexpr int kPlanSmallTiles = 4, kPlanBigParts = 5, kPlanSmallParts = 6, kPlanMerged = 7;
//         [12] row tiles of height bm1 in buckets of several, if the buckets of one are at least as many (mixed_tile in ffn_tiles.h); else 0
constexpr int kPlanLateUp = 8, kPlanLateDown = 9, kPlanOwnBegin = 10, kPlanOwnEnd = 11, kPlanMixed = 12;

// Merged buckets.  On the receive side an expert's rows arrive as one segment per source GPU.  As buckets of their own
// they stream the expert's weights once per segment and end in a ragged tile each, so segments of one expert form one
// bucket whose rows are numbered through.  kPlanStart then holds the bucket's first entry in the segment list; entry j
// says that the bucket's rows from kPlanSegOff[j] on lie at kPlanSegDelta[j] + row.  The first segment of a bucket, and
// only that, begins at row 0, and so does the entry past the last one: that is how a walk along the list ends.
struct RowMap {
    bool merged;             // false: the rows follow each other
    int row0;                // buffer row of row 0 of the tile (not merged)
    int first, last;         // the tile's rows within the bucket
    int delta;               // of the segment that holds `first`
    int more;                // segments after that one that hold rows of the tile, at most 64 of them in ...
    int off_lane, delta_lane;    // ... the wavefront's lanes
    const int32_t* rest;     // entry after those 64 (more == 64)
};

// the map of rows first .. first + rows - 1 of the listed bucket whose kPlanStart entry is `start`; called by whole
// wavefronts, which fetch the bucket's segments together: one round of memory latency instead of one per segment and row
__device__ __forceinline__ RowMap row_map_at(const int32_t* __restrict__ plan, int start, bool merged, int first, int rows) {
    RowMap m;
    m.merged = merged;
    m.row0 = start + first;
    m.first = first;
    m.last = first + rows - 1;
    m.more = m.off_lane = m.delta_lane = m.delta = 0;
    m.rest = nullptr;
    if (!m.merged) return m;
    const int32_t* off = plan + kPlanSegOff;
    const int lane = threadIdx.x & 63;
    int seg = start;
    for (;;) {                                            // skip the segments before the one that holds `first`
        const int o = off[min(seg + 1 + lane, MOE_MAX_EXPERTS)];
        const unsigned long long stop = __ballot(o == 0 || o > first);
        seg += stop ? __builtin_ctzll(stop) : 64;
        if (stop) break;
    }
    const int j = min(seg + 1 + lane, MOE_MAX_EXPERTS);
    m.off_lane = off[j];
    m.delta_lane = plan[kPlanSegDelta + min(j, MOE_MAX_EXPERTS - 1)];
    m.delta = plan[kPlanSegDelta + seg];
    const unsigned long long stop = __ballot(m.off_lane == 0 || m.off_lane > m.last || j != seg + 1 + lane);
    m.more = stop ? __builtin_ctzll(stop) : 64;
    m.rest = off + seg + 65;
    return m;
}
// ... of listed bucket i (MAY_MERGE = false: the caller knows that nothing is merged)
template <bool MAY_MERGE>
__device__ __forceinline__ RowMap row_map(const int32_t* __restrict__ plan, int i, int first, int rows) {
    return row_map_at(plan, plan[kPlanStart + i], MAY_MERGE && plan[kPlanMerged], first, rows);
}

// Where row r of the tile lies in the buffer (0 <= r < rows).  It reads the segments out of other lanes' registers, so
// the whole wavefront calls it, outside any branch that only some lanes take (there the compiler may refill or copy a
// register for the active lanes only): a store to a ragged tile clamps its row, asks for the address and then decides
// whether to store.
__device__ __forceinline__ int buffer_row(const RowMap& m, int r) {
    if (!m.merged) return m.row0 + r;
    const int b = m.first + r;
    int at = m.delta;
    for (int j = 0; j < m.more; ++j) {
        const int o = __builtin_amdgcn_readlane(m.off_lane, j), d = __builtin_amdgcn_readlane(m.delta_lane, j);
        at = b >= o ? d : at;
    }
    if (m.more == 64)                                     // many tiny segments: the rest of the list from memory
        for (const int32_t* p = m.rest; *p != 0 && *p <= m.last; ++p) at = b >= *p ? p[kPlanSegDelta - kPlanSegOff] : at;
    return at + b;
}

// E groups of rows (counts/starts); group g multiplies with the weights of expert group_expert[g]
// (g itself when group_expert is NULL), of which there are n_weights; placement may be NULL when
// local_gpu < 0.
// choice: 0 or 1 fixes header [3]; -1 lets the device decide from the listed buckets: bm0 when they hold
// at least kLargeBucketRows rows on average, else bm1.
constexpr int kLargeBucketRows = 544;     // measured crossover at the Mixtral shape: 512 rows per bucket favour 256-row tiles by 1 %, 640 favour 384 by 5 %
// merge: what becomes of several groups with the same weights: 0 each stays a bucket, 1 they are merged, 2 they are
// merged unless the groups are large enough for the tall tiles as they are; with merge_shape.cpx > 0 only where
// merge_pays (1: the streaming kernels follow, 2: the tiled ones)
int launch_ffn_plan(const int32_t* counts, const int32_t* starts, const int32_t* placement, int local_gpu,
                    const int32_t* group_expert, int n_weights, int E, int N, const PlanShape& shape, int merge, const MergeShape& merge_shape,
                    int32_t* plan, hipStream_t s);

constexpr int kF32TileRows = 32, kF32SplitRows = 64;    // tile heights of the fp32 path: small batches, large ones
constexpr int kTallTileRows = 384, kShortTileRows = 256; // tile heights of the bf16 path
constexpr int kSkinnyRows = 64;                         // rows a pass of its streaming kernels covers (bm1 of their plan)

// kPlanMixed of a plan of `tiles` row tiles of which `single` are buckets of one (mixed_tile in ffn_tiles.h: why the line lies there)
__host__ __device__ __forceinline__ int mixed_rows(int tiles, int single) { return 2 * single >= tiles ? tiles - single : 0; }

// The plan's counts in one word, so that one LDS operation adds a group to all: groups with rows, those of one row tile of bm1, those whose
// last tile has at most kSmallTileRows rows (up to 256 each, 9 bits), and row tiles of bm1 (fewer than 2^31 / kF32TileRows + 256, 27 bits).
struct PlanSums {
    unsigned long long v;
    static __device__ __forceinline__ unsigned long long of(int tiles, bool single, bool small) {
        return ((unsigned long long)tiles << 27) | ((unsigned)small << 18) | ((unsigned)single << 9) | 1u;
    }
    __device__ __forceinline__ int listed() const { return (int)v & 511; }
    __device__ __forceinline__ int single() const { return (int)(v >> 9) & 511; }
    __device__ __forceinline__ int small() const { return (int)(v >> 18) & 511; }
    __device__ __forceinline__ int tiles() const { return (int)(v >> 27); }
};

// Shared memory of build_plan: per group its rows and tiles, and the sums over the groups listed before it.
struct PlanScratch {
    int cnt[MOE_MAX_EXPERTS], tiles0[MOE_MAX_EXPERTS], tiles1[MOE_MAX_EXPERTS], segs[MOE_MAX_EXPERTS];
    int rank[MOE_MAX_EXPERTS], rows[MOE_MAX_EXPERTS], pre0[MOE_MAX_EXPERTS], pre1[MOE_MAX_EXPERTS], pre_segs[MOE_MAX_EXPERTS];
    unsigned long long sums;                             // four counts in one word (PlanSums)
    int first_row[MOE_MAX_EXPERTS / 64];                 // of the groups of a wavefront with rows (only when the range of all is asked for)
};

// The cut of a one-round launch, for the plan's header; called by one wavefront, a lane per candidate.
__device__ __forceinline__ void round_split(int lane, int nb, int ns, const PlanShape& shape, int32_t* __restrict__ plan) {
    const RoundShape r = round_shape(nb, ns, shape.nt_down, shape.kt_down, shape.cus_per_xcd);
    RoundCut best = round_candidate(r, lane % kRoundCandidates);
    static_assert(kRoundCandidates == 16, "the lanes of one DPP row");
    const auto across = [&](auto ctrl) {                   // the better one of this lane's and the other half of its group's
        const int cost = __builtin_amdgcn_mov_dpp(best.cost, decltype(ctrl)::value, 0xF, 0xF, true);
        const int how = __builtin_amdgcn_mov_dpp(best.big | best.small << 8 | best.rounds << 16, decltype(ctrl)::value, 0xF, 0xF, true);
        best = better_cut(best, {cost, how & 255, how >> 8 & 255, how >> 16});
    };
    across(std::integral_constant<int, 0xB1>());           // neighbours, pairs, ...
    across(std::integral_constant<int, 0x4E>());
    across(std::integral_constant<int, 0x141>());          // ... halves of eight and the row mirrored: a half agrees by then
    across(std::integral_constant<int, 0x140>());
    if (best.big == 0) {                                   // wave-uniform
        if (lane == 0) plan[kPlanBigParts] = 0;
        return;
    }
    const RoundCut even = even_cut(r);
    const bool odd = lane & 1;                             // even lanes price the cut, odd ones the even split
    const float cost = launch_cost(r, odd ? even.big : best.big, odd ? even.small : best.small, odd ? even.rounds : best.rounds);
    const float other = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, cost), 0xB1, 0xF, 0xF, true));
    if (lane == 0) {
        plan[kPlanBigParts] = cost < other + kSearchCost ? best.big : 0;
        plan[kPlanSmallParts] = best.small;
    }
}

// Builds the plan with one workgroup of at least MOE_MAX_EXPERTS threads (a whole power of two), all of which must
// call this: thread e brings group e's row count c (0: not listed; threads past the last group bring 0), its first
// row st and the expert wt whose weights it multiplies with; with `merged`, group e is a merged bucket of n_segs
// segments and its rank and place in the segment list are left in the scratch; range: the range of rows of all groups, which is
// contiguous, is wanted in the header.  The E x E comparisons are dealt to all
// threads (thread: group, slice of the others); walked by one thread per group they took 5.5 us for E = 64.
__device__ __forceinline__ void build_plan(PlanScratch& s, int e, int c, int st, int wt, int E, const PlanShape& shape,
                                           int32_t* __restrict__ plan, bool merged = false, int n_segs = 0, bool range = false) {
    if (e < MOE_MAX_EXPERTS) {
        s.cnt[e] = c;
        s.tiles0[e] = (c + shape.bm0 - 1) / shape.bm0;
        s.tiles1[e] = (c + shape.bm1 - 1) / shape.bm1;
        s.segs[e] = n_segs;
        s.rank[e] = s.rows[e] = s.pre0[e] = s.pre1[e] = s.pre_segs[e] = 0;
    }
    if (e == 0) s.sums = 0;
    if (range && e < MOE_MAX_EXPERTS) {                  // the groups with rows lie side by side, by number
        const unsigned long long some = __ballot(c > 0);
        if ((e & 63) == (some ? __builtin_ctzll(some) : 0)) s.first_row[e >> 6] = some ? st : 0x7FFFFFFF;
    }
    __syncthreads();
    // One LDS operation.  Four sums, one of them of different values and so, as the compiler has it, a loop over the lanes / ballots and
    // exchanges per wavefront / this, us: 64 experts, top-6, front of 64 tokens 10.2 / 8.5 / 8.4, one-workgroup kernel of 2000 16.3 /
    // 14.8 / 14.6, plan of 64 received segments 5.3 / 5.8 / 5.3; front of 1000 fp32 tokens, 8 experts, whose weights have swept the kernel's
    // instructions out of the caches, 9.5 / 10.1 / 9.4.
    if (c > 0) {
        const int tiles = s.tiles1[e];
        int at = 0;
        asm("" : "+v"(at));                              // could differ by lane, for all the compiler knows: no loop
        atomicAdd(&s.sums + at, PlanSums::of(tiles, c <= shape.bm1, c - (tiles - 1) * shape.bm1 <= kSmallTileRows));
    }
    int ebits = 0;
    while ((1 << ebits) < E) ++ebits;
    const int EP = 1 << ebits, me = e & (EP - 1), slices = (int)blockDim.x >> ebits;
    int r = 0, rows = 0, t0 = 0, t1 = 0, sg = 0;
    if (me < E && s.cnt[me] > 0) {
        const int mine = s.cnt[me];
#pragma unroll 4
        for (int o = e >> ebits; o < E; o += slices) {
            const int co = s.cnt[o], a = s.tiles0[o], b = s.tiles1[o], g = s.segs[o];
            const bool first = (co > mine) | ((co == mine) & (o < me));       // false for a group without rows
            r += first;
            rows += first ? co : 0;
            t0 += first ? a : 0;
            t1 += first ? b : 0;
            sg += first ? g : 0;
        }
    }
    for (int m = EP; m < 64; m <<= 1) {
        r += __shfl_xor(r, m, 64);
        rows += __shfl_xor(rows, m, 64);
        t0 += __shfl_xor(t0, m, 64);
        t1 += __shfl_xor(t1, m, 64);
        sg += __shfl_xor(sg, m, 64);
    }
    if (me < E && (e & 63) < EP) {
        atomicAdd(&s.rank[me], r);
        atomicAdd(&s.rows[me], rows);
        atomicAdd(&s.pre0[me], t0);
        atomicAdd(&s.pre1[me], t1);
        atomicAdd(&s.pre_segs[me], sg);
    }
    __syncthreads();
    const PlanSums sums = {s.sums};
    const int n = sums.listed(), n_small = sums.small();
    if (c > 0) {
        r = s.rank[e];
        t0 = s.pre0[e];
        t1 = s.pre1[e];
        plan[kPlanExpert + r] = wt;
        plan[kPlanStart + r] = merged ? s.pre_segs[e] : st;
        plan[kPlanCount + r] = c;
        plan[kPlanTiles0 + r] = t0;
        plan[kPlanTiles1 + r] = t1;
        if (r == n - 1) {                                // the last listed group knows the totals
            t0 += s.tiles0[e];
            t1 += s.tiles1[e];
            plan[0] = n;
            plan[1] = t0;
            plan[2] = t1;
            const int choice = shape.choice >= 0 ? shape.choice : ((long long)s.rows[e] + c >= (long long)kLargeBucketRows * n ? 0 : 1);
            plan[3] = choice;
            plan[kPlanSmallTiles] = 1 + n_small;
            plan[kPlanMerged] = merged;
            plan[kPlanMixed] = mixed_rows(t1, sums.single());
            plan[kPlanTiles0 + n] = t0;
            plan[kPlanTiles1 + n] = t1;
            if (range) {
                int begin = s.first_row[0];
#pragma unroll
                for (int w = 1; w < MOE_MAX_EXPERTS / 64; ++w) begin = min(begin, s.first_row[w]);
                plan[kPlanOwnBegin] = begin;
                plan[kPlanOwnEnd] = begin + s.rows[e] + c;
            }
        }
    } else if (n == 0 && e == 0) {
        plan[0] = plan[1] = plan[2] = plan[kPlanMerged] = plan[kPlanMixed] = 0;
        plan[3] = shape.choice >= 0 ? shape.choice : 0;
        plan[kPlanSmallTiles] = 1;
        plan[kPlanTiles0] = plan[kPlanTiles1] = 0;
        if (range) plan[kPlanOwnBegin] = plan[kPlanOwnEnd] = 0;
    }
    const int last_wave = (int)blockDim.x - 64;          // while the others write
    if (e >= last_wave) {
        if (shape.kt_down > 0) round_split(e - last_wave, sums.tiles() - n_small, n_small, shape, plan);
        else if (e == last_wave) plan[kPlanBigParts] = 0;
    }
}

}  // namespace moe
