// moe_topk_gate: top-k router (paper Section 2.1).
//
// Which lanes and lists serve how many experts; the selection itself is in
// gate_select.h.  A token's E logits are spread over L neighbouring lanes of a
// wavefront in pieces of four, VPL logits per lane (16-byte loads when
// E % 4 == 0), so a wavefront reads 64/L whole rows, neighbouring lanes
// neighbouring pieces.  Up to 8 experts one lane scans its token's keys in k
// rounds; above, every lane sorts its candidates into a list of KMAX >= k and the
// lists are merged across the lanes.  Weights are the softmax over the k selected
// logits in fp32, or (ALL) the softmax over all E logits read at the selected
// experts.
#include "gate_select.h"

namespace moe {

template <int L, int VPL, int KMAX, bool ALL, bool FULL>
__global__ __launch_bounds__(256) void gate_kernel(const float* __restrict__ logits, int T, int E, int k,
                                                   int32_t* __restrict__ topk_idx, float* __restrict__ topk_w) {
    constexpr int TOK_PER_BLOCK = 256 / L;
    const int sub = threadIdx.x % L;
    const long long t = (long long)blockIdx.x * TOK_PER_BLOCK + threadIdx.x / L;
    const bool live = t < T;
    gate_select<L, VPL, KMAX, ALL, FULL>(logits + (live ? t : 0) * E, false, sub, live, t, E, k, topk_idx, topk_w);
}

template <int L, int VPL, bool ALL, bool FULL>
static void launch_k(const float* logits, int T, int E, int k, int32_t* idx, float* w, hipStream_t s) {
    constexpr int TOK_PER_BLOCK = 256 / L;
    const unsigned grid = (unsigned)(((long long)T + TOK_PER_BLOCK - 1) / TOK_PER_BLOCK);
    if (k <= 2) hipLaunchKernelGGL((gate_kernel<L, VPL, 2, ALL, FULL>), dim3(grid), dim3(256), 0, s, logits, T, E, k, idx, w);
    else if (L == 1 || k <= 8) hipLaunchKernelGGL((gate_kernel<L, VPL, 8, ALL, FULL>), dim3(grid), dim3(256), 0, s, logits, T, E, k, idx, w);      // one lane: E <= 8
    else hipLaunchKernelGGL((gate_kernel<L, VPL, L == 1 ? 8 : MOE_MAX_TOPK, ALL, FULL>), dim3(grid), dim3(256), 0, s, logits, T, E, k, idx, w);
}

// whether every lane holds as many logits as it can is known here (FULL in gate_select.h); one lane alone asks anyway
template <int L, int VPL, bool ALL>
static void launch_l(const float* logits, int T, int E, int k, int32_t* idx, float* w, hipStream_t s) {
    if (L > 1 && E == L * VPL) launch_k<L, VPL, ALL, (L > 1)>(logits, T, E, k, idx, w, s);
    else launch_k<L, VPL, ALL, false>(logits, T, E, k, idx, w, s);
}

template <bool ALL>
static void launch_e(const float* logits, int T, int E, int k, int32_t* idx, float* w, hipStream_t s) {
    if (E <= 4) launch_l<1, 4, ALL>(logits, T, E, k, idx, w, s);
    else if (E <= 8) launch_l<1, 8, ALL>(logits, T, E, k, idx, w, s);
    else if (E <= 16) launch_l<2, 8, ALL>(logits, T, E, k, idx, w, s);
    else if (E <= 32) launch_l<4, 8, ALL>(logits, T, E, k, idx, w, s);
    else if (E <= 64) launch_l<4, 16, ALL>(logits, T, E, k, idx, w, s);
    else if (E <= 128) launch_l<8, 16, ALL>(logits, T, E, k, idx, w, s);
    else launch_l<16, 16, ALL>(logits, T, E, k, idx, w, s);
}

int launch_gate(const float* logits, int T, int E, int k, bool all_norm, int32_t* idx, float* w, hipStream_t s) {
    LaunchTimer timer(MOE_K_GATE, s);
    if (all_norm) launch_e<true>(logits, T, E, k, idx, w, s);
    else launch_e<false>(logits, T, E, k, idx, w, s);
    return check_launch("moe_topk_gate launch");
}

}  // namespace moe
