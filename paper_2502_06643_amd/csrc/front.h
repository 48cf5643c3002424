// The fused front of moe_layer_forward (front.hip): gate, dispatch and tile plan in one launch.
#pragma once
#include "common.h"

namespace moe {

constexpr int kFrontMaxRoutes = 12288;   // routes a workgroup sorts by itself (their expert ids fill 24 KB of LDS)
constexpr int kFrontGroups = 256;        // workgroups: one per compute unit, all but the first two with at least one token
constexpr int kFrontMaxPasses = 6;       // passes of the gate, of one token per thread
constexpr long long kFrontMaxBytes = 72ll << 20; // of the send rows
constexpr int kFrontMaxTokens = 25;      // tokens a workgroup may own (front_fits keeps T within what the others own)

struct FrontArgs {
    const uint4* x;                      // [T] rows of units_per_row 16-byte pieces
    const float* logits;
    int T, E, k, G, local_gpu, units_per_row, ebits;
    const int32_t* placement;
    int32_t *topk_idx, *perm, *inv_perm, *expert_counts, *expert_start, *gpu_counts, *gpu_offsets;
    float* topk_w;
    uint4* send_buf;
    PlanShape shape;                     // of the tile plan
    int32_t* plan;
};

bool front_fits(int T, int E, int k, int row_bytes);
int launch_front(const FrontArgs& a, hipStream_t s);

}  // namespace moe
