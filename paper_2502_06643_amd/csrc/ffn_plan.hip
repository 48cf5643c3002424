#include "ffn_plan.h"

namespace moe {

constexpr int kPlanThreads = 1024;
__global__ __launch_bounds__(kPlanThreads) void ffn_plan_kernel(const int32_t* __restrict__ counts, const int32_t* __restrict__ starts,
                                                       const int32_t* __restrict__ placement, int local_gpu,
                                                       const int32_t* __restrict__ group_expert, int n_weights, int E, int N,
                                                       int bm0, int bm1, int choice, int32_t* __restrict__ plan) {
    __shared__ PlanScratch scratch;
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
    build_plan(scratch, e, c, st, wt, E, bm0, bm1, choice, plan);
}

PlanShape ffn_plan_shape(moe_dtype_t dt, int N, int E, bool every_row_resident) {
    if (dt == MOE_F32) return {kF32TileRows, kF32TileRows, 0};
    if (N <= kFfnSkinnyMaxRows) return {kShortTileRows, kShortTileRows, 0};
    // Row tiles of 384 move about a sixth fewer bytes per flop than tiles of 256, but waste more on
    // ragged buckets and leave compute units idle when there are few tiles: 384 when the resident buckets
    // hold kLargeBucketRows rows or more on average.  When every row is in a resident bucket the host
    // knows that average; otherwise only the device does and the plan decides.  Either way the choice
    // reaches the kernels through the plan's header.
    const int choice = every_row_resident ? ((long long)N >= (long long)kLargeBucketRows * E ? 0 : 1) : -1;
    return {kTallTileRows, kShortTileRows, choice};
}

int launch_ffn_plan(const int32_t* counts, const int32_t* starts, const int32_t* placement, int local_gpu,
                    const int32_t* group_expert, int n_weights, int E, int N, const PlanShape& shape, int32_t* plan, hipStream_t s) {
    LaunchTimer timer(MOE_K_FFN_PLAN, s);
    hipLaunchKernelGGL(ffn_plan_kernel, dim3(1), dim3(kPlanThreads), 0, s, counts, starts, placement, local_gpu, group_expert, n_weights, E, N,
                       shape.bm0, shape.bm1, shape.choice, plan);
    return check_launch("moe_expert_ffn_grouped plan launch");
}

}  // namespace moe
