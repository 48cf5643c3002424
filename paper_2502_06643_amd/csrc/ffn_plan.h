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
constexpr int kPlanInts = kPlanTiles1 + MOE_MAX_EXPERTS + 4;
static_assert(kPlanInts * sizeof(int32_t) <= kPlanBytes, "plan area too small");
// header: [0] number of listed experts, [1] total row tiles (bm0), [2] total row tiles (bm1),
//         [3] which of the two tile heights the bf16 GEMMs use: 0 = bm0, 1 = bm1 (see `choice`)

// E groups of rows (counts/starts); group g multiplies with the weights of expert group_expert[g]
// (g itself when group_expert is NULL), of which there are n_weights; placement may be NULL when
// local_gpu < 0.
// choice: 0 or 1 fixes header [3]; -1 lets the device decide from the listed buckets: bm0 when they hold
// at least kLargeBucketRows rows on average, else bm1.
constexpr int kLargeBucketRows = 544;     // measured crossover at the Mixtral shape: 512 rows per bucket favour 256-row tiles by 1 %, 640 favour 384 by 5 %
int launch_ffn_plan(const int32_t* counts, const int32_t* starts, const int32_t* placement, int local_gpu,
                    const int32_t* group_expert, int n_weights, int E, int N, const PlanShape& shape, int32_t* plan, hipStream_t s);

constexpr int kF32TileRows = 32;                        // tile height of the fp32 path
constexpr int kTallTileRows = 384, kShortTileRows = 256; // tile heights of the bf16 path

// Shared memory of build_plan: per group its rows and tiles, and the sums over the groups listed before it.
struct PlanScratch {
    int cnt[MOE_MAX_EXPERTS], tiles0[MOE_MAX_EXPERTS], tiles1[MOE_MAX_EXPERTS];
    int rank[MOE_MAX_EXPERTS], rows[MOE_MAX_EXPERTS], pre0[MOE_MAX_EXPERTS], pre1[MOE_MAX_EXPERTS];
};

// Builds the plan with one workgroup of at least MOE_MAX_EXPERTS threads (a whole power of two), all of which must
// call this: thread e brings group e's row count c (0: not listed; threads past the last group bring 0), its first
// row st and the expert wt whose weights it multiplies with.  The E x E comparisons are dealt to all threads
// (thread: group, slice of the others); walked by one thread per group they took 5.5 us for E = 64.
__device__ __forceinline__ void build_plan(PlanScratch& s, int e, int c, int st, int wt, int E, int bm0, int bm1, int choice,
                                           int32_t* __restrict__ plan) {
    if (e < MOE_MAX_EXPERTS) {
        s.cnt[e] = c;
        s.tiles0[e] = (c + bm0 - 1) / bm0;
        s.tiles1[e] = (c + bm1 - 1) / bm1;
        s.rank[e] = s.rows[e] = s.pre0[e] = s.pre1[e] = 0;
    }
    const int n = __syncthreads_count(c > 0);
    int ebits = 0;
    while ((1 << ebits) < E) ++ebits;
    const int EP = 1 << ebits, me = e & (EP - 1), slices = (int)blockDim.x >> ebits;
    int r = 0, rows = 0, t0 = 0, t1 = 0;
    if (me < E && s.cnt[me] > 0) {
        const int mine = s.cnt[me];
#pragma unroll 4
        for (int o = e >> ebits; o < E; o += slices) {
            const int co = s.cnt[o], a = s.tiles0[o], b = s.tiles1[o];
            const bool first = (co > mine) | ((co == mine) & (o < me));       // false for a group without rows
            r += first;
            rows += first ? co : 0;
            t0 += first ? a : 0;
            t1 += first ? b : 0;
        }
    }
    for (int m = EP; m < 64; m <<= 1) {
        r += __shfl_xor(r, m, 64);
        rows += __shfl_xor(rows, m, 64);
        t0 += __shfl_xor(t0, m, 64);
        t1 += __shfl_xor(t1, m, 64);
    }
    if (me < E && (e & 63) < EP) {
        atomicAdd(&s.rank[me], r);
        atomicAdd(&s.rows[me], rows);
        atomicAdd(&s.pre0[me], t0);
        atomicAdd(&s.pre1[me], t1);
    }
    __syncthreads();
    if (c > 0) {
        r = s.rank[e];
        t0 = s.pre0[e];
        t1 = s.pre1[e];
        plan[kPlanExpert + r] = wt;
        plan[kPlanStart + r] = st;
        plan[kPlanCount + r] = c;
        plan[kPlanTiles0 + r] = t0;
        plan[kPlanTiles1 + r] = t1;
        if (r == n - 1) {                                // the last listed group knows the totals
            t0 += s.tiles0[e];
            t1 += s.tiles1[e];
            plan[0] = n;
            plan[1] = t0;
            plan[2] = t1;
            plan[3] = choice >= 0 ? choice : ((long long)s.rows[e] + c >= (long long)kLargeBucketRows * n ? 0 : 1);
            plan[kPlanTiles0 + n] = t0;
            plan[kPlanTiles1 + n] = t1;
        }
    } else if (n == 0 && e == 0) {
        plan[0] = plan[1] = plan[2] = 0;
        plan[3] = choice >= 0 ? choice : 0;
        plan[kPlanTiles0] = plan[kPlanTiles1] = 0;
    }
}

}  // namespace moe
