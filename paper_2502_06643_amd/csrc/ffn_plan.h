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
#include "common.h"

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
constexpr int kPlanSmallTiles = 4, kPlanBigParts = 5, kPlanSmallParts = 6, kPlanMerged = 7;
constexpr int kSmallTileRows = 128;

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

// the map of rows first .. first + rows - 1 of listed bucket i; called by whole wavefronts, which fetch the bucket's
// segments together: one round of memory latency instead of one per segment and row
// (MAY_MERGE = false: the caller knows that nothing is merged)
template <bool MAY_MERGE>
__device__ __forceinline__ RowMap row_map(const int32_t* __restrict__ plan, int i, int first, int rows) {
    RowMap m;
    const int start = plan[kPlanStart + i];
    m.merged = MAY_MERGE && plan[kPlanMerged];
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
// merged unless the groups are large enough for the tall tiles as they are
int launch_ffn_plan(const int32_t* counts, const int32_t* starts, const int32_t* placement, int local_gpu,
                    const int32_t* group_expert, int n_weights, int E, int N, const PlanShape& shape, int merge, int32_t* plan,
                    hipStream_t s);

constexpr int kF32TileRows = 32;                        // tile height of the fp32 path
constexpr int kTallTileRows = 384, kShortTileRows = 256; // tile heights of the bf16 path
constexpr int kSkinnyRows = 64;                         // rows a pass of its streaming kernels covers (bm1 of their plan)

// Shared memory of build_plan: per group its rows and tiles, and the sums over the groups listed before it.
struct PlanScratch {
    int cnt[MOE_MAX_EXPERTS], tiles0[MOE_MAX_EXPERTS], tiles1[MOE_MAX_EXPERTS], segs[MOE_MAX_EXPERTS];
    int rank[MOE_MAX_EXPERTS], rows[MOE_MAX_EXPERTS], pre0[MOE_MAX_EXPERTS], pre1[MOE_MAX_EXPERTS], pre_segs[MOE_MAX_EXPERTS];
    int n, n_small, total1;
};

// Split of a down projection whose 256-row tiles all run in one round (at most one tile per compute unit).  The launch
// then lasts as long as its longest tile, so tiles are cut along k by what they cost: a tile of more than kSmallTileRows
// rows into `big` parts, the others into `small`.  A k tile takes 1.3 us in the former (bound by the matrix pipes and
// its 64 KB) and about 1 us in the latter (bound by its weight stream).  777 tokens at the Mixtral shape are 80 such
// tiles and 96 small ones, 176 on 256 compute units: 312 us with the fix-up uncut, 275 with the 80 cut in two.
// kSplitCost and kPartCost stand for the partial tiles' way through memory and the fix-up (10 us and 1.3 us a part;
// twice and half of that chose about as well).  Called by one wavefront: lane (rounds, b) tries one or two rounds of parts (two fp32 partial tiles exist per compute
// unit) with the big tiles in b parts.
constexpr int kXcds = 8;
constexpr int kMaxSplit = 8;
constexpr int kMinSplitKT = 8;                  // a k part is at least this many k tiles
constexpr int kMinSplitGain = 16;               // k tiles of time a split tail must save to be worth its fix-up
// whether any split of a reduction of KT k tiles can save that much
constexpr bool split_can_pay(int KT) {
    const int parts = KT / kMinSplitKT < kMaxSplit ? KT / kMinSplitKT : kMaxSplit;
    return parts > 1 && (KT - KT / parts) >= kMinSplitGain;
}
__device__ __forceinline__ void round_split(int lane, int nb, int ns, const PlanShape& shape, int32_t* __restrict__ plan) {
    constexpr int kBigCost = 4, kSmallCost = 3, kSplitCost = 32, kPartCost = 4;
    const int KT = shape.kt_down, cpx = shape.cus_per_xcd, q = shape.nt_down / kXcds, rem = shape.nt_down % kXcds;
    const int nbx = nb * q + (nb * rem + kXcds - 1) / kXcds, nsx = ns * q + (ns * rem + kXcds - 1) / kXcds;     // the fullest XCD
    const int whole = (nbx > 0 ? kBigCost : kSmallCost) * KT;
    int best = whole, big = 0, small = 1;
    if (nbx + nsx > 0 && nbx + nsx <= cpx) {
        const int rounds = 1 + lane / kMaxSplit % 2, b = 1 + lane % kMaxSplit;
        const int left = rounds * cpx - b * nbx;
        if (left >= nsx && (b == 1 || (nbx > 0 && KT / b >= kMinSplitKT))) {
            const int tb = nbx > 0 ? kBigCost * ((KT + b - 1) / b) : 0;
            // the small tiles in as many parts as it takes not to outlast the big ones, as far as there is room
            int sm = 1;
            if (nsx > 0) {
                sm = tb > 0 ? (kSmallCost * KT + tb - 1) / tb : kMaxSplit;
                sm = min(min(sm, kMaxSplit), min(left / nsx, KT / kMinSplitKT));
                sm = max(sm, 1);
            }
            const int ts = nsx > 0 ? kSmallCost * ((KT + sm - 1) / sm) : 0, t = rounds * (tb > ts ? tb : ts);
            // ... and what the partial tiles and the fix-up cost, in the same unit of a third of a microsecond
            const int parts = max(b, sm), cost = t + kSplitCost + kPartCost * parts;
            if (parts > 1 && cost < whole) { best = cost; big = b; small = sm; }
        }
        for (int m = 1; m < 2 * kMaxSplit; m <<= 1) {             // the shortest, then the fewest parts
            const int ot = __shfl_xor(best, m, 64), ob = __shfl_xor(big, m, 64), os = __shfl_xor(small, m, 64);
            if (ot < best || (ot == best && ob + os < big + small)) { best = ot; big = ob; small = os; }
        }
    }
    if (lane == 0) {
        plan[kPlanBigParts] = big;
        plan[kPlanSmallParts] = small;
    }
}

// Builds the plan with one workgroup of at least MOE_MAX_EXPERTS threads (a whole power of two), all of which must
// call this: thread e brings group e's row count c (0: not listed; threads past the last group bring 0), its first
// row st and the expert wt whose weights it multiplies with; with `merged`, group e is a merged bucket of n_segs
// segments and its rank and place in the segment list are left in the scratch.  The E x E comparisons are dealt to all
// threads (thread: group, slice of the others); walked by one thread per group they took 5.5 us for E = 64.
__device__ __forceinline__ void build_plan(PlanScratch& s, int e, int c, int st, int wt, int E, const PlanShape& shape,
                                           int32_t* __restrict__ plan, bool merged = false, int n_segs = 0) {
    if (e < MOE_MAX_EXPERTS) {
        s.cnt[e] = c;
        s.tiles0[e] = (c + shape.bm0 - 1) / shape.bm0;
        s.tiles1[e] = (c + shape.bm1 - 1) / shape.bm1;
        s.segs[e] = n_segs;
        s.rank[e] = s.rows[e] = s.pre0[e] = s.pre1[e] = s.pre_segs[e] = 0;
    }
    if (e == 0) s.n = s.n_small = s.total1 = 0;
    __syncthreads();
    if (c > 0) {
        atomicAdd(&s.n, 1);
        atomicAdd(&s.total1, s.tiles1[e]);
        if (c - (s.tiles1[e] - 1) * shape.bm1 <= kSmallTileRows) atomicAdd(&s.n_small, 1);
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
    const int n = s.n, n_small = s.n_small;
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
            plan[3] = shape.choice >= 0 ? shape.choice : ((long long)s.rows[e] + c >= (long long)kLargeBucketRows * n ? 0 : 1);
            plan[kPlanSmallTiles] = 1 + n_small;
            plan[kPlanMerged] = merged;
            plan[kPlanTiles0 + n] = t0;
            plan[kPlanTiles1 + n] = t1;
        }
    } else if (n == 0 && e == 0) {
        plan[0] = plan[1] = plan[2] = plan[kPlanMerged] = 0;
        plan[3] = shape.choice >= 0 ? shape.choice : 0;
        plan[kPlanSmallTiles] = 1;
        plan[kPlanTiles0] = plan[kPlanTiles1] = 0;
    }
    const int last_wave = (int)blockDim.x - 64;          // while the others write
    if (e >= last_wave) {
        if (shape.kt_down > 0) round_split(e - last_wave, s.total1 - n_small, n_small, shape, plan);
        else if (e == last_wave) plan[kPlanBigParts] = 0;
    }
}

}  // namespace moe
