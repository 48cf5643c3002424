#include "ffn_late.h"

namespace moe {

constexpr int kPlanThreads = 1024;

struct MergeScratch {
    int wt[MOE_MAX_EXPERTS], cnt[MOE_MAX_EXPERTS];           // per group
    int off[MOE_MAX_EXPERTS], idx[MOE_MAX_EXPERTS];          // ... its first row and its number among its bucket's segments
    int rows[MOE_MAX_EXPERTS], segs[MOE_MAX_EXPERTS];        // per expert
    int pays;
};

__global__ __launch_bounds__(kPlanThreads) void ffn_plan_kernel(const int32_t* __restrict__ counts, const int32_t* __restrict__ starts,
                                                                const int32_t* __restrict__ placement, int local_gpu,
                                                                const int32_t* __restrict__ group_expert, int n_weights, int E, int N,
                                                                PlanShape shape, int merge, MergeShape merge_shape, int32_t* __restrict__ plan) {
    __shared__ PlanScratch scratch;
    __shared__ MergeScratch ms;
    const int e = threadIdx.x;
    int c = 0, st = 0, wt = e;                    // wt: whose weights this group multiplies with
    if (e < E) {
        const bool local = local_gpu < 0 || placement[e] == local_gpu;
        c = counts[e];
        st = starts[e];
        if (group_expert) wt = group_expert[e];
        // a bucket that does not lie inside [0,N), or names weights that do not exist, is ignored rather than trusted
        if (!local || c <= 0 || st < 0 || (long long)st + c > N || (unsigned)wt >= (unsigned)n_weights) c = 0;
    }
    int n = 0;                                    // groups with rows
    if (merge != 0) {
        if (e < MOE_MAX_EXPERTS) {
            ms.wt[e] = wt;
            ms.cnt[e] = c;
            ms.off[e] = ms.idx[e] = ms.rows[e] = ms.segs[e] = 0;
        }
        n = __syncthreads_count(c > 0);
        if (c > 0) {
            atomicAdd(&ms.rows[wt], c);
            atomicAdd(&ms.segs[wt], 1);
        }
        __syncthreads();
        const int n_buckets = __syncthreads_count(e < MOE_MAX_EXPERTS && ms.segs[e & (MOE_MAX_EXPERTS - 1)] > 0);
        if (n_buckets == n) merge = 0;
        if (merge != 0 && e < 64) {
            // One wavefront adds everything up and decides: sums of different values into one LDS address go lane by lane,
            // 3 to 5 us for 64 segments
            const int bm1_bits = __builtin_ctz(shape.bm1);    // 32, 64 or 256 rows
            int total = 0;
            Buckets apart = {0, 0}, merged = {0, 0};
#pragma unroll
            for (int i = 0; i < MOE_MAX_EXPERTS / 64; ++i) {
                const int co = ms.cnt[i * 64 + e], ro = ms.rows[i * 64 + e];
                total += co;
                apart = {apart.tiles + ((co + shape.bm1 - 1) >> bm1_bits), max(apart.max_rows, co)};
                merged = {merged.tiles + ((ro + shape.bm1 - 1) >> bm1_bits), max(merged.max_rows, ro)};
            }
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) {
                total += __shfl_xor(total, m, 64);
                apart = {apart.tiles + __shfl_xor(apart.tiles, m, 64), max(apart.max_rows, __shfl_xor(apart.max_rows, m, 64))};
                merged = {merged.tiles + __shfl_xor(merged.tiles, m, 64), max(merged.max_rows, __shfl_xor(merged.max_rows, m, 64))};
            }
            const bool pays = !(merge == 2 && total >= (long long)kLargeBucketRows * n) &&
                              (merge_shape.cpx == 0 || merge_pays(merge_shape, apart, merged, merge == 1));
            if (e == 0) ms.pays = pays;
        }
        __syncthreads();
        if (merge != 0 && !ms.pays) merge = 0;
    }
    if (merge == 0) {
        build_plan(scratch, e, c, st, wt, E, shape, plan);
        return;
    }
    // rows and segments of the same expert in the groups before mine: thread (group, slice of the groups)
    int ebits = 0;
    while ((1 << ebits) < E) ++ebits;
    const int EP = 1 << ebits, me = e & (EP - 1);
    int off = 0, idx = 0;
    if (me < E) {
        const int w = ms.wt[me];
        for (int o = e >> ebits; o < me; o += kPlanThreads >> ebits) {
            const int co = ms.cnt[o];
            const bool same = ms.wt[o] == w && co > 0;
            off += same ? co : 0;
            idx += same;
        }
    }
    for (int m = EP; m < 64; m <<= 1) {
        off += __shfl_xor(off, m, 64);
        idx += __shfl_xor(idx, m, 64);
    }
    if (me < E && (e & 63) < EP) {
        atomicAdd(&ms.off[me], off);
        atomicAdd(&ms.idx[me], idx);
    }
    if (merge == 2) shape.choice = 1;             // the kernels of the short tiles know how to follow the segments
    const bool expert = e < n_weights;
    build_plan(scratch, e, expert ? ms.rows[e] : 0, 0, e, n_weights, shape, plan, true, expert ? ms.segs[e] : 0);
    if (c > 0) {
        const int j = scratch.pre_segs[wt] + ms.idx[e];
        plan[kPlanSegOff + j] = ms.off[e];
        plan[kPlanSegDelta + j] = st - ms.off[e];
    }
    if (e == 0) plan[kPlanSegOff + n] = 0;        // (a count here instead waited for the stores: 0.7 to 1.9 us)
}

// Which bf16 batches run the weight-streaming kernels: up to kFfnSkinnyMaxRows routes all of them (measured at that limit), and
// up to kMaxRows those that make few tasks of the up projection however the routes fall: at most one chunk of rows per expert and
// one more per 64 routes.  Such a launch is one round of tasks that are all cut, and the tiled kernels' is all latency: staging
// and barriers of a few k tiles, with rows for a fraction of a tile, and a fix-up launch.  What decides otherwise is how
// many experts the routes reach and how evenly, which the host does not know (nor what is resident, so that this
// does not depend on it): 129 to 255 tasks are neither cut nor two to a compute unit, and a bucket of many chunks reads its weights
// once for each.  Measured on random layers of 161 to 900 routes, 1 to 128 experts of 0.02 M to 16 M (d f), all or a part of them
// resident, uniform to all at one (34000): inside 11706, 0.99 to 2.6 times as fast, 1.46 on average; with up to 128 tasks the worst
// is 0.89, with up to 159 0.84.  Layer, us, tiled / streaming: 8 experts, 320 routes, d 768, f 576 38 / 29; 32, 390, d 1280, f 192 40 / 38; 8, 559, d
// 2368, f 768 65 / 65.  Outside: 8 of 64 experts, 640 skewed routes, d 4096, f 3584 199 / 270; all of 64, 161 routes, d 2048, f 1408 71 / 81,
// 584, 537 of them at one expert, 80 / 92; 128, 224 routes, d 1472, f 768 52 / 69; but 8 of 64, 360 routes, d 2048, f 1408 55 / 29.
bool ffn_streams(int N, int d, int f, int E, bool segments) {
    constexpr int kMaxRows = 640, kMaxTasks = 96, kMaxHidden = 4096;
    if (N <= kFfnSkinnyMaxRows) return true;
    const long long tasks = (long long)((E < N ? E : N) + N / kSkinnyRows) * ((f + 127) / 128);
    return !segments && N <= kMaxRows && d <= kMaxHidden && tasks <= kMaxTasks;
}

int ffn_plan_shape(moe_dtype_t dt, int N, int d, int f, int E, bool every_row_resident, bool segments, PlanShape* shape) {
    *shape = {kF32TileRows, kF32SplitRows, 0, 0, 0, 0};
    if (dt == MOE_F32) return MOE_OK;
    shape->bm0 = kShortTileRows;
    shape->bm1 = kSkinnyRows;
    if (ffn_streams(N, d, f, E, segments)) return MOE_OK;
    shape->bm1 = kShortTileRows;
    // Row tiles of 384 move about a sixth fewer bytes per flop than tiles of 256, but waste more on
    // ragged buckets and leave compute units idle when there are few tiles: 384 when the resident buckets
    // hold kLargeBucketRows rows or more on average.  When every row is in a resident bucket the host
    // knows that average; otherwise only the device does and the plan decides.  Either way the choice
    // reaches the kernels through the plan's header.
    shape->bm0 = kTallTileRows;
    shape->choice = every_row_resident ? ((long long)N >= (long long)kLargeBucketRows * E ? 0 : 1) : -1;
    shape->nt_down = (d + 255) / 256;
    shape->kt_down = split_can_pay(f / 64) ? f / 64 : 0;
    return ffn_bf16_device_setup(&shape->cus_per_xcd);
}

// The tiled bf16 kernels only; the down projection takes rows where none of its tiles is cut along k to fill the chip.  How
// many tiles this GPU has, and so how many rows it can copy beside them, only the device knows (late_tokens).  Not asked about:
// calls that with an even routing have an eighth more than a round of tiles (where the rows of a GPU's experts are few, the routing decides; the
// question itself costs 0.2 %); rows of less than kMinBytes for others, which are copied before the projections by the time
// that these have slowed down (175 random layers of 8 to 48 MB 1.003 times as fast, the worst 0.976, of 80 MB and more see
// ffn_late.h); reductions of fewer k tiles than kMinKTiles, whose tiles are over before the copies are under way (d 960, f 960, 16 experts,
// top-4, 6719 tokens 100.8 us, with late rows 102); and up to two routes a token, because its row is read once more (21 random layers
// 0.997 times as fast in the median, the worst 0.99; with three 43 layers 1.037, the worst 0.99).
LateShape ffn_late_shape(moe_dtype_t dt, int N, int d, int f, int E, int T, int k, int G, int cus_per_xcd) {
    constexpr long long kMinBytes = 80ll << 20;
    constexpr int kMinKTiles = 20, kMinRoutes = 3;
    LateShape l = {};
    if (dt != MOE_BF16 || G < 2 || k < kMinRoutes || d / 64 < kMinKTiles || ffn_streams(N, d, f, E, false)) return l;
    const long long row_tiles = N / G / kShortTileRows > E / G ? N / G / kShortTileRows : E / G;
    if (row_tiles * ((f + 127) / 128) >= 9ll * cus_per_xcd || (long long)(N - N / G) * d * 2 < kMinBytes) return l;
    const float per_kt = (float)kXcds * (float)kLateBytesPerKTile / ((float)d * 2.0f);
    l.nt_up = (f + 127) / 128;
    l.nt_down = (d + 255) / 256;
    l.rows_up = per_kt * (float)(d / 64);
    l.rows_down = split_can_pay(f / 64) ? 0.f : per_kt * (float)(f / 64);
    l.per_token = 1.0f / (float)T;
    l.cus_per_xcd = cus_per_xcd;
    l.T = T;
    l.k = k;
    return l;
}

int launch_ffn_plan(const int32_t* counts, const int32_t* starts, const int32_t* placement, int local_gpu,
                    const int32_t* group_expert, int n_weights, int E, int N, const PlanShape& shape, int merge, const MergeShape& merge_shape,
                    int32_t* plan, hipStream_t s) {
    LaunchTimer timer(MOE_K_FFN_PLAN, s);
    hipLaunchKernelGGL(ffn_plan_kernel, dim3(1), dim3(kPlanThreads), 0, s, counts, starts, placement, local_gpu, group_expert, n_weights, E, N,
                       shape, merge, merge_shape, plan);
    return check_launch("moe_expert_ffn_grouped plan launch");
}

}  // namespace moe
