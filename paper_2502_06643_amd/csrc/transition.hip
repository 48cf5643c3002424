// moe_transition_counts: the layer-l -> layer-(l+1) routing history table
// R_{e1,e2,l} of the paper (Section 2.4; Section 3.1 "Token Routing Profile";
// ILP 2 inputs).
//
// Each workgroup keeps private int32 copies of the E_l x E_l1 table in LDS
// (as many copies as fit, up to 32, selected by lane so that lanes hitting the
// same hot bin mostly land on different addresses), counts its tokens'
// k_l * k_l1 expert pairs (or only its top-1 pair) there with LDS atomics, and then adds its non-zero
// bins to the int64 table in memory.  Integer adds commute, so the result is
// exact whatever the order.  A table too large for LDS is cut into stripes of
// rows: a workgroup counts one stripe only.
#include "common.h"

namespace moe {

constexpr int kTransThreads = 1024;
constexpr int kLdsBins = 12288;          // 48 KB of int32: two workgroups fit a compute unit
constexpr int kLdsBinsLarge = 32768;     // 128 KB: one does, with a 128 x 256 table
constexpr int kTokPerThread = 4;

// rows: table rows of one stripe (blockIdx.y counts the stripes)
template <int LDS_BINS>
__global__ __launch_bounds__(kTransThreads) void transition_kernel(const int32_t* __restrict__ idx_l, const int32_t* __restrict__ idx_l1,
                                                         int T, int k_l, int k_l1, int use_l, int use_l1, int E_l, int E_l1, int rows,
                                                         int copies, int pairs_of_two, unsigned long long* __restrict__ R) {
    __shared__ __attribute__((aligned(16))) int hist[LDS_BINS];
    const int row0 = blockIdx.y * rows, rows_here = min(rows, E_l - row0), bins = rows_here * E_l1;
    const int my_copy = threadIdx.x & (copies - 1);
    for (int b = threadIdx.x * 4; b < bins * copies; b += kTransThreads * 4) *reinterpret_cast<int4*>(hist + b) = make_int4(0, 0, 0, 0);
    __syncthreads();
    const long long stride = (long long)gridDim.x * kTransThreads;
    auto count = [&](int e1, int e2) {
        if ((unsigned)(e1 - row0) >= (unsigned)rows_here || (unsigned)e2 >= (unsigned)E_l1) return;
        atomicAdd(&hist[((e1 - row0) * E_l1 + e2) * copies + my_copy], 1);
    };
    long long t = (long long)blockIdx.x * kTransThreads + threadIdx.x;
    if (pairs_of_two) {
        // top-2 in both layers (the usual case) and 8-byte aligned arrays: 8-byte loads, eight tokens per thread in flight at a time
        const int2* a2 = reinterpret_cast<const int2*>(idx_l);
        const int2* b2 = reinterpret_cast<const int2*>(idx_l1);
        auto count_pairs = [&](int2 a, int2 b) {
            count(a.x, b.x);
            if (use_l1 > 1) count(a.x, b.y);
            if (use_l > 1) {
                count(a.y, b.x);
                if (use_l1 > 1) count(a.y, b.y);
            }
        };
        for (; t + 7 * stride < T; t += 8 * stride) {
            int2 a[8], b[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) { a[u] = a2[t + u * stride]; b[u] = b2[t + u * stride]; }
#pragma unroll
            for (int u = 0; u < 8; ++u) count_pairs(a[u], b[u]);
        }
        for (; t < T; t += 4 * stride) {                   // the tail: slots past the batch hold -1, which count() ignores
            int2 a[4], b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool in = t + u * stride < T;
                a[u] = in ? a2[t + u * stride] : make_int2(-1, -1);
                b[u] = in ? b2[t + u * stride] : make_int2(-1, -1);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) count_pairs(a[u], b[u]);
        }
    }
    if (use_l <= 8 && use_l1 <= 8) {
        // up to 8 x 8 pairs per token: both index lists go to registers first (all loads in flight together;
        // slots past use_l / use_l1 hold -1, which count() ignores)
        for (; t < T; t += stride) {
            int e1s[8], e2s[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                e1s[j] = j < use_l ? idx_l[t * k_l + j] : -1;
                e2s[j] = j < use_l1 ? idx_l1[t * k_l1 + j] : -1;
            }
#pragma unroll
            for (int j1 = 0; j1 < 8; ++j1) {
                if (j1 >= use_l) break;
#pragma unroll
                for (int j2 = 0; j2 < 8; ++j2) count(e1s[j1], e2s[j2]);
            }
        }
    }
    for (; t < T; t += stride) {
        for (int j1 = 0; j1 < use_l; ++j1) {              // the first use_l of the k_l slots (all of them, or the top-1)
            const int e1 = idx_l[t * k_l + j1];
            for (int j2 = 0; j2 < use_l1; ++j2)
                count(e1, idx_l1[t * k_l1 + j2]);         // re-read per pair: it stays in L1, and no private array is needed
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < bins; b += kTransThreads) {
        int c = 0;
        for (int i = 0; i < copies; ++i) c += hist[b * copies + ((i + threadIdx.x) & (copies - 1))];
        if (c) atomicAdd(&R[(size_t)row0 * E_l1 + b], (unsigned long long)c);
    }
}

int launch_transition(const int32_t* idx_l, const int32_t* idx_l1, int T, int k_l, int k_l1, int E_l, int E_l1,
                      bool top1_only, int64_t* R, hipStream_t s) {
    const int use_l = top1_only ? 1 : k_l, use_l1 = top1_only ? 1 : k_l1;
    const int pairs_of_two = k_l == 2 && k_l1 == 2 && ((uintptr_t)idx_l & 7) == 0 && ((uintptr_t)idx_l1 & 7) == 0;
    const bool large = E_l * E_l1 > kLdsBins;
    const int rows = large && E_l * E_l1 > kLdsBinsLarge ? kLdsBinsLarge / E_l1 : E_l;
    const int stripes = (E_l + rows - 1) / rows, bins = rows * E_l1;
    // tokens per thread: four for top-2 x top-2, one when a token has 16 pairs or more
    const int pairs = use_l * use_l1;
    const int tpt = pairs >= 16 ? 1 : (pairs >= 8 ? 2 : kTokPerThread);
    // Every workgroup ends with one global atomic per non-zero bin, all workgroups on the same lines, so their number is
    // kept at 128 of 1024 threads.  Measured with 512 / 256 / 128 / 64 workgroups: 4 M tokens, 8 experts, top-2 19.4 / 16.1
    // / 15.2 / 21.1 us; 100003 tokens, 64 experts, top-6 8.8 / 8.7 / 8.7 / 11.1 (15.6 with 391 workgroups of 256 threads);
    // 65536 tokens, 128 experts, top-8 15.2 / 15.2 / 15.4 / 15.4.  Batches of a few thousand tokens do not care.  Tables of
    // more than 110 x 110 used to be counted straight into memory: 32768 tokens, 128 experts, top-8 1177 us, now 14.4.
    constexpr long long cap = 128;
    const long long want = ((long long)T + (long long)kTransThreads * tpt - 1) / ((long long)kTransThreads * tpt);
    const dim3 grid((unsigned)(want < 1 ? 1 : (want > cap ? cap : want)), (unsigned)stripes);
    int copies = 1;
    while (copies < 32 && bins * copies * 2 <= kLdsBins) copies *= 2;
    LaunchTimer timer(MOE_K_TRANSITION, s);
    if (large)
        hipLaunchKernelGGL(transition_kernel<kLdsBinsLarge>, grid, dim3(kTransThreads), 0, s, idx_l, idx_l1, T, k_l, k_l1, use_l, use_l1,
                           E_l, E_l1, rows, copies, pairs_of_two, (unsigned long long*)R);
    else
        hipLaunchKernelGGL(transition_kernel<kLdsBins>, grid, dim3(kTransThreads), 0, s, idx_l, idx_l1, T, k_l, k_l1, use_l, use_l1,
                           E_l, E_l1, rows, copies, pairs_of_two, (unsigned long long*)R);
    return check_launch("moe_transition_counts launch");
}

}  // namespace moe
