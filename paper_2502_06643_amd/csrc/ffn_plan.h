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

// Shared memory of build_plan, four entries per expert slot.
struct PlanScratch {
    __attribute__((aligned(16))) int cnt[MOE_MAX_EXPERTS];
    __attribute__((aligned(16))) int rank[MOE_MAX_EXPERTS];
    __attribute__((aligned(16))) int tiles0[MOE_MAX_EXPERTS];
    __attribute__((aligned(16))) int tiles1[MOE_MAX_EXPERTS];
};

// Builds the plan with one workgroup of at least MOE_MAX_EXPERTS threads, all of which must call this: thread e
// brings group e's row count c (0: not listed; threads past the last group bring 0), its first row st and the
// expert wt whose weights it multiplies with.
__device__ __forceinline__ void build_plan(PlanScratch& s, int e, int c, int st, int wt, int E, int bm0, int bm1, int choice,
                                           int32_t* __restrict__ plan) {
    if (e < MOE_MAX_EXPERTS) {
        s.cnt[e] = c;
        s.tiles0[e] = (c + bm0 - 1) / bm0;
        s.tiles1[e] = (c + bm1 - 1) / bm1;
    }
    __syncthreads();
    // the loops below read the shared arrays four entries at a time; entries from E on hold zeros / -1
    const int E4 = (E + 3) / 4;
    int r = 0;
    if (c > 0) {
        const int4* cnt4 = reinterpret_cast<const int4*>(s.cnt);
        for (int q = 0; q < E4; ++q) {
            const int4 co = cnt4[q];
            const int o = 4 * q;
            r += ((co.x > c) | ((co.x == c) & (o < e))) + ((co.y > c) | ((co.y == c) & (o + 1 < e))) +
                 ((co.z > c) | ((co.z == c) & (o + 2 < e))) + ((co.w > c) | ((co.w == c) & (o + 3 < e)));
        }
    }
    if (e < MOE_MAX_EXPERTS) s.rank[e] = (c > 0) ? r : -1;
    __syncthreads();
    if (c > 0) {
        int t0 = 0, t1 = 0;
        const int4* rank4 = reinterpret_cast<const int4*>(s.rank);
        const int4* tl0 = reinterpret_cast<const int4*>(s.tiles0);
        const int4* tl1 = reinterpret_cast<const int4*>(s.tiles1);
        for (int q = 0; q < E4; ++q) {
            const int4 ro = rank4[q], a = tl0[q], b = tl1[q];
            const bool k0 = (ro.x >= 0) & (ro.x < r), k1 = (ro.y >= 0) & (ro.y < r), k2 = (ro.z >= 0) & (ro.z < r), k3 = (ro.w >= 0) & (ro.w < r);
            t0 += (k0 ? a.x : 0) + (k1 ? a.y : 0) + (k2 ? a.z : 0) + (k3 ? a.w : 0);
            t1 += (k0 ? b.x : 0) + (k1 ? b.y : 0) + (k2 ? b.z : 0) + (k3 ? b.w : 0);
        }
        plan[kPlanExpert + r] = wt;
        plan[kPlanStart + r] = st;
        plan[kPlanCount + r] = c;
        plan[kPlanTiles0 + r] = t0;
        plan[kPlanTiles1 + r] = t1;
    }
    if (e == 0) {
        int n = 0, t0 = 0, t1 = 0;
        long long rows = 0;
        const int4* cnt4 = reinterpret_cast<const int4*>(s.cnt);
        const int4* tl0 = reinterpret_cast<const int4*>(s.tiles0);
        const int4* tl1 = reinterpret_cast<const int4*>(s.tiles1);
        for (int q = 0; q < E4; ++q) {
            const int4 co = cnt4[q], a = tl0[q], b = tl1[q];
            n += (co.x > 0) + (co.y > 0) + (co.z > 0) + (co.w > 0);
            rows += (long long)co.x + co.y + co.z + co.w;
            t0 += a.x + a.y + a.z + a.w;
            t1 += b.x + b.y + b.z + b.w;
        }
        plan[0] = n;
        plan[1] = t0;
        plan[2] = t1;
        plan[3] = choice >= 0 ? choice : (rows >= (long long)kLargeBucketRows * n ? 0 : 1);
        plan[kPlanTiles0 + n] = t0;
        plan[kPlanTiles1 + n] = t1;
    }
}

}  // namespace moe
