// The front of a layer in one launch: gate (moe_topk_gate), dispatch (moe_dispatch) and the tile plan of the expert
// FFN, for batches small enough that a workgroup can route all of them by itself (paper Section 2.1, Section 2.2,
// Section 3.1).
//
// At these sizes each of the four launches it replaces takes 4.5-10 us, nearly all of it launch latency.  Here every
// workgroup works out the whole batch's routing redundantly - gate into LDS, the counting sort of the routes - and
// then writes only its own share: the gate outputs, positions and send rows of its tokens.  Workgroups 0 and 1 have no
// tokens: the one writes the tile plan, the other the expert and GPU tables.  Nothing passes between workgroups.  The first pieces
// of the workgroup's rows are loaded before anything else, so that they arrive while it routes.
#include "dispatch_index.h"
#include "ffn_plan.h"
#include "gate_select.h"
#include "front.h"

namespace moe {

constexpr int kFrontTableGroups = 2;     // workgroups without tokens
constexpr int kFrontPrefetch = 4;        // 16-byte pieces of x per thread that are loaded up front

template <int L, int VPL, int KMAX>
__global__ __launch_bounds__(kIndexThreads) void front_kernel(FrontArgs a) {
    __shared__ IndexTables s;
    __shared__ PlanScratch plan_scratch;
    __shared__ uint16_t ids[kFrontMaxRoutes];              // expert of every route
    __shared__ int my_pos[kFrontMaxTokens * MOE_MAX_TOPK]; // positions of this workgroup's routes
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    const int T = a.T, E = a.E, k = a.k, N = T * k;
    const int groups = gridDim.x - kFrontTableGroups, g = (int)blockIdx.x - kFrontTableGroups;
    const int t0 = g < 0 ? T : (int)((long long)g * T / groups), t1 = g < 0 ? T : (int)((long long)(g + 1) * T / groups);
    const int units = (t1 - t0) * a.units_per_row;
    const uint4* rows = a.x + (long long)t0 * a.units_per_row;
    uint4 pre[kFrontPrefetch];
#pragma unroll
    for (int i = 0; i < kFrontPrefetch; ++i) {
        const int u = tid + i * kIndexThreads;
        pre[i] = u < units ? rows[u] : make_uint4(0u, 0u, 0u, 0u);
    }
    index_clear(s, E);
    if (tid < E) s.pl[tid] = a.placement[tid];

    // gate: L lanes per token, the whole batch; one copy of the selection, which asks which logits exist (FULL in gate_select.h)
    const int sub = tid % L;
    for (int base = 0; base < T; base += kIndexThreads / L) {
        const int t = base + tid / L;
        const bool live = t < T;
        constexpr int S = kGateSlots<L, KMAX>;
        gate_select_emit<L, VPL, KMAX, false, false>(a.logits + (long long)(live ? t : 0) * E, false, sub, live, E, k,
                                              [&](const int (&e_sel)[S], const float (&p_sel)[S], float denom) {
#pragma unroll
                                                  for (int i = 0; i < S; ++i)
                                                      if (sub + L * i < k) ids[t * k + sub + L * i] = (uint16_t)e_sel[i];
                                                  if (t >= t0 && t < t1) gate_store<L, S>(t, sub, k, e_sel, p_sel, denom, a.topk_idx, a.topk_w);
                                              });
    }
    __syncthreads();

    // the counting sort: every wavefront counts its slice of the routes ...
    const int per_wave = ((N + kIndexThreads - 1) / kIndexThreads) * 64, wbase = wave * per_wave, wend = min(N, wbase + per_wave);
    const unsigned long long lower = (1ull << lane) - 1ull;
    for (int r0 = wbase; r0 < wend; r0 += 64) {
        const int r = r0 + lane, ex = r < wend ? ids[r] : MOE_MAX_EXPERTS;
        const bool ok = ex < E;
        const unsigned long long m = match_expert(ex, ok, a.ebits);
        if (ok && (m & lower) == 0ull) atomicAdd(&s.woff[wave][ex], __popcll(m));       // first lane of the group
    }
    __syncthreads();
    index_totals(s, E, a.ebits);
    if (blockIdx.x == 0) {
        int c = 0, st = 0;
        if (tid < E && (a.local_gpu < 0 || s.pl[tid] == a.local_gpu)) {
            c = s.tot[tid];
            st = s.start[tid];
        }
        build_plan(plan_scratch, tid, c, st, tid, E, a.shape, a.plan);
        return;
    }
    if (blockIdx.x == 1) {
        index_write_tables(s, E, a.G, a.expert_counts, a.expert_start, a.gpu_counts, a.gpu_offsets);
        return;
    }
    // ... and walks it as far as this workgroup's own routes reach
    const int own0 = t0 * k, own1 = t1 * k;
    if (wbase < own1 && own0 < wend) {
        for (int r0 = wbase; r0 < min(wend, own1); r0 += 64) {
            const int r = r0 + lane, ex = r < wend ? ids[r] : MOE_MAX_EXPERTS;
            const bool ok = ex < E;
            const int pos = index_next(s.woff[wave], ex, ok, a.ebits, lower);
            if (r >= own0 && r < own1) {
                my_pos[r - own0] = ok ? pos : -1;
                if (ok) {
                    a.perm[pos] = r;
                    a.inv_perm[r] = pos;
                }
            }
        }
    }
    __syncthreads();

    // rows: every 16-byte piece was or is read once and is written to its token's k positions
    auto put = [&](int u, const uint4& v) {
        const int t = u / a.units_per_row, c = u - t * a.units_per_row;
        for (int j = 0; j < k; ++j) {
            const int p = my_pos[t * k + j];
            if ((unsigned)p < (unsigned)N) a.send_buf[(long long)p * a.units_per_row + c] = v;
        }
    };
#pragma unroll
    for (int i = 0; i < kFrontPrefetch; ++i) {
        const int u = tid + i * kIndexThreads;
        if (u < units) put(u, pre[i]);
    }
    for (int u = tid + kFrontPrefetch * kIndexThreads; u < units; u += kIndexThreads) put(u, rows[u]);
}

// lanes per token of the gate for E experts
static int front_lanes(int E) { return E <= 8 ? 1 : (E <= 64 ? 4 : 16); }

bool front_fits(int T, int E, int k, int row_bytes) {
    // Every workgroup gates and sorts the whole batch by itself, which is what the launches it saves are worth only for so
    // many passes of the gate: six with one lane per token, with more lanes (sorted lists) two up to top-2 and one beyond.
    // And one workgroup a compute unit copies rows slower than a launch of its own, which shows past kFrontMaxBytes of them.
    // Layer with a small FFN, us, separate launches / fused: 8 experts, top-2, d 4096, 4096 tokens (67 MB of rows) 157 / 156,
    // 6144 (101 MB) 182 / 186; fp32, d 256, 6144 tokens (13 MB) 48.1 / 46.8; top-1, d 2048, 6144 tokens 96.2 / 95.2, 8192 102 / 103;
    // 64 experts, top-2, d 1024, 512 tokens 46.5 / 45.2, 768 48.8 / 50.6; 64 experts, top-6, d 2048, 256 tokens 68.7 / 66.0,
    // 512 72.1 / 72.3, 2048 115 / 137; 128 experts, top-8, d 1024, 64 tokens 46.2 / 44.0, 128 50.7 / 51.8, 512 64 / 86; 256
    // experts, top-2, d 2048, 128 tokens 72.8 / 71.9, 256 75.2 / 79.4.
    const long long N = (long long)T * k;
    const int passes = front_lanes(E) == 1 ? kFrontMaxPasses : (k <= 2 ? 2 : 1);
    static_assert(kFrontMaxPasses * kIndexThreads <= (kFrontGroups - kFrontTableGroups) * kFrontMaxTokens, "a workgroup's tokens fit its tables");
    return T > 0 && N <= kFrontMaxRoutes && N * row_bytes <= kFrontMaxBytes && (long long)T * front_lanes(E) <= (long long)passes * kIndexThreads;
}

template <int L, int VPL>
static void launch_lanes(const FrontArgs& a, int grid, hipStream_t s) {
    if (a.k <= 2) hipLaunchKernelGGL((front_kernel<L, VPL, 2>), dim3(grid), dim3(kIndexThreads), 0, s, a);
    else if (L == 1 || a.k <= 8) hipLaunchKernelGGL((front_kernel<L, VPL, 8>), dim3(grid), dim3(kIndexThreads), 0, s, a);      // one lane: E <= 8
    else hipLaunchKernelGGL((front_kernel<L, VPL, L == 1 ? 8 : MOE_MAX_TOPK>), dim3(grid), dim3(kIndexThreads), 0, s, a);
}

int launch_front(const FrontArgs& args, hipStream_t s) {
    FrontArgs a = args;
    a.ebits = 0;
    while ((1 << a.ebits) < a.E) ++a.ebits;
    const int grid = a.T < kFrontGroups - kFrontTableGroups ? a.T + kFrontTableGroups : kFrontGroups;
    LaunchTimer timer(MOE_K_FRONT, s);
    switch (front_lanes(a.E)) {
        case 1: launch_lanes<1, 8>(a, grid, s); break;
        case 4: launch_lanes<4, 16>(a, grid, s); break;
        default: launch_lanes<16, 16>(a, grid, s); break;
    }
    return check_launch("moe_layer_forward front launch");
}

}  // namespace moe
