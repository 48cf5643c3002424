// moe_router_gate: the linear router in front of the top-k gate (paper Section
// 2.1): logits = x . W_g + bias and moe_topk_gate's selection on them, in ONE
// kernel: the logits of a workgroup's tokens never leave the compute unit
// (writing them to memory is optional).
//
// bf16: a skinny GEMM on the matrix cores that is bound by reading x once.  A
// workgroup owns up to 32 tokens; its wavefronts (4 to 16, see below) split the
// reduction into contiguous shares, each feeding v_mfma_f32_32x32x16_bf16 with the activation
// fragment (lane l: token l % 32, 8 consecutive k; fetched as whole lines and
// re-ordered through a staging tile in LDS, see the kernel) and the
// weight fragments from the pre-packed router matrix (moe_pack_router: for every
// 16 reduction steps and every 32 experts one 1 KB block in B-fragment order, so
// a fragment is one coalesced 16-byte load per lane).  The partial sums are
// added through LDS in wavefront order, so results are reproducible; the 32 x E
// logits stay in LDS (and go to memory when asked to) and 256 threads run the
// gate's selection on them, 8 lanes per token.
// fp32: one workgroup per token, one thread per expert, sequential fp32 sum,
// then 16 lanes select from the row in LDS.
#include "gate_select.h"
#include <type_traits>

namespace moe {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

static inline int padded_experts(int E) { return (E + 31) / 32 * 32; }

size_t router_packed_bytes(int d, int E, moe_dtype_t dt) {
    return dt == MOE_BF16 ? (size_t)padded_experts(E) * d * 2 : (size_t)d * E * sizeof(float);
}

// unit o = (kb * panels + panel) * 64 + lane holds 8 consecutive k of one expert column
__global__ __launch_bounds__(256) void pack_router_bf16_kernel(const uint16_t* __restrict__ w_g, int d, int E, int panels,
                                                               long long total, uint4* __restrict__ packed) {
    const long long o = (long long)blockIdx.x * 256 + threadIdx.x;
    if (o >= total) return;
    const int lane = (int)(o & 63);
    const long long blk = o >> 6;
    const int panel = (int)(blk % panels);
    const int kb = (int)(blk / panels);
    const int e = panel * 32 + (lane & 31);
    const int k0 = kb * 16 + 8 * (lane >> 5);
    uint16_t v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (e < E) ? w_g[(size_t)(k0 + i) * E + e] : (uint16_t)0;
    uint4 q;
    q.x = v[0] | ((uint32_t)v[1] << 16); q.y = v[2] | ((uint32_t)v[3] << 16);
    q.z = v[4] | ((uint32_t)v[5] << 16); q.w = v[6] | ((uint32_t)v[7] << 16);
    packed[o] = q;
}

int launch_pack_router(const void* w_g, int d, int E, moe_dtype_t dt, void* packed, hipStream_t s) {
    if (dt == MOE_F32) {
        hipError_t e = hipMemcpyAsync(packed, w_g, (size_t)d * E * sizeof(float), hipMemcpyDeviceToDevice, s);
        return e == hipSuccess ? MOE_OK : hip_fail(e, "moe_pack_router copy");
    }
    const int panels = padded_experts(E) / 32;
    const long long total = (long long)(d / 16) * panels * 64;
    hipLaunchKernelGGL(pack_router_bf16_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, (const uint16_t*)w_g, d, E,
                       panels, total, (uint4*)packed);
    return check_launch("moe_pack_router launch");
}

// LDS of the bf16 kernel, in floats: a staging tile of 32 tokens x 64 k (bf16) per wavefront, then the partial sums
// [PANELS][16][64] (sixteen wavefronts: [16][16][64] of one panel), then the logits [32 tokens]
// [32 * PANELS + 4] (rows padded by 16 bytes), one after the other in the same memory
constexpr int router_lds_floats(int panels, int waves) {
    const int stage = waves * 32 * 64 / 2, sums = (waves == 4 ? panels : waves) * 16 * 64, rows = 32 * (32 * panels + 4);
    return stage > sums ? (stage > rows ? stage : rows) : (sums > rows ? sums : rows);
}

// WAVES wavefronts share the reduction, whose chain of k steps, each at the latency of memory, is all there is to a small
// batch; with several workgroups on a compute unit the read of x is what bounds the launch (launch_router_gate has the rule).
// Four / eight / sixteen, us: 8 experts, d 4096, 64 tokens 8.3 / 7.5 / 7.3, 4096 10.8 / 9.1 / 12.1, 6000 12.0 / 11.1 / 13.6,
// 8192 14.1 / 17.7 / 18.8, 24000 39 / 44 / 50, d 2048, 10007 tokens 10.8 / 10.1 / 15.6; 64 experts, d 4096, 2048 tokens 21 /
// 13.8 / 13.6, 8192 25.0 / 19.7 / 22.9, d 2048, 16384 20.8 / 18.6 / 23.9, 24000 31 / 37 / 35; 128 experts, d 4096, 2048 tokens
// 34 / 26 / 20, 24000 90 / 87 / 87, 65536 207 / 186 / 232, d 1024, 65536 75 / 63 / 81.
// AHEAD (one panel): the weights are fetched through a buffer descriptor, one stage ahead, and the activations two.
template <int PANELS, int KMAX, int WAVES, bool AHEAD>
__global__ __launch_bounds__(64 * WAVES, WAVES == 8 && PANELS > 2 ? 4 : 1) void router_gate_bf16_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ packed,
                                                               const float* __restrict__ bias, int T, int d, int E, int k,
                                                               float* __restrict__ logits, int32_t* __restrict__ topk_idx,
                                                               float* __restrict__ topk_w, int tokens) {
    extern __shared__ __attribute__((aligned(16))) float red[];      // activation staging, then [PANELS][16][64] partial sums, then the logits
    const int lane = threadIdx.x & 63, wave = WAVES == 4 ? (int)(threadIdx.x >> 6) : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar with four: 17.4 -> 20.6 us at 10007 tokens
    const long long t0 = (long long)blockIdx.x * tokens, last = min(t0 + tokens, (long long)T) - 1;
    const uint16_t* wlane = packed + (size_t)lane * 8;
    f32x16 acc[PANELS];
#pragma unroll
    for (int p = 0; p < PANELS; ++p)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[p][v] = 0.f;
    // Each wavefront owns a contiguous share of the reduction and streams it in stages of 64 k: 32 tokens x
    // 128 bytes, fetched as four fully coalesced 16-byte loads per lane (lane l: token 8 j + l / 8, 16-byte chunk
    // l % 8: whole 128-byte lines) into registers one stage ahead, written to a staging tile of its own in LDS
    // (no barrier: a wavefront's LDS accesses execute in order) whose eight 16-byte slots per row are XOR-swizzled
    // by (row >> 1) & 7, and read back as the A operand of the matrix instruction (lane l: token l % 32, the 8
    // consecutive k that start at 8 * (l / 32) of every 16): conflict-free both ways.  Loading the operand
    // straight from memory instead costs four partly used lines per instruction.
    constexpr int KSTAGE = 64;
    uint16_t* stage = reinterpret_cast<uint16_t*>(red) + wave * (32 * KSTAGE);
    // this wavefront's k: whole steps of 16; what is left of the last stage of 64 goes the direct way
    const int kw0 = WAVES == 4 ? wave * (d / 4) : (int)((long long)wave * (d / 16) / WAVES) * 16;
    const int KSW = WAVES == 4 ? d / 4 : (int)((long long)(wave + 1) * (d / 16) / WAVES) * 16 - kw0;
    const int n_stage = KSW / KSTAGE;
    if constexpr (AHEAD) {
        static_assert(PANELS == 1, "one block of weights a step");
        // Loads return in order, so a stage's weights are asked for one stage ahead and before the activations of the stage
        // after that, two ahead: waiting for one stage leaves the next one's activations in flight.  With the weights asked for
        // in the stage that needs them, behind the next stage's activations, every stage waited for both: 65536 tokens, d 4096,
        // 8 experts 106 us, now 97.
        u32x4 xr[3][4], wr[2][4];
        const int lr = lane >> 3, lc = lane & 7;
        const uint16_t* xl[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) xl[j] = x + min(t0 + 8 * j + lr, last) * d + kw0 + lc * 8;       // tokens past the workgroup's re-read its last one
        auto fetch_x = [&](int st, u32x4 (&r)[4]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) r[j] = *reinterpret_cast<const u32x4*>(xl[j] + st * KSTAGE);
        };
        // lanes whose expert does not exist point past the descriptor: they move no bytes and get the zeros that stand there
        const auto wsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(packed), 0, 32 * d * 2, 0x00020000);
        const uint32_t woff = (lane & 31) < E ? (uint32_t)(kw0 / 16 * 64 + lane) * 16u : 0x80000000u;
        auto fetch_w = [&](int st, u32x4 (&r)[4]) {
#pragma unroll
            for (int u = 0; u < 4; ++u) r[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wsrc, woff + (uint32_t)((st * 4 + u) * 1024), 0, 0));
        };
        auto multiply = [&](const u32x4 (&xs)[4], const u32x4 (&ws)[4]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int row = 8 * j + lr;
                *reinterpret_cast<u32x4*>(stage + row * KSTAGE + ((lc ^ ((row >> 1) & 7)) * 8)) = xs[j];
            }
#pragma unroll
            for (int u = 0; u < KSTAGE / 16; ++u) {
                const int row = lane & 31;
                const bf16x8 a = *reinterpret_cast<const bf16x8*>(stage + row * KSTAGE + (((2 * u + (lane >> 5)) ^ ((row >> 1) & 7)) * 8));
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, ws[u]), acc[0], 0, 0, 0);
            }
        };
        if (n_stage > 0) {
            fetch_x(0, xr[0]);
            fetch_w(0, wr[0]);
            fetch_x(min(1, n_stage - 1), xr[1]);
            for (int st = 0; st < n_stage; st += 6) {    // buffers by stage number; past the end the last stage is fetched again
#pragma unroll
                for (int u = 0; u < 6; ++u) {
                    fetch_w(min(st + u + 1, n_stage - 1), wr[(u + 1) & 1]);
                    fetch_x(min(st + u + 2, n_stage - 1), xr[(u + 2) % 3]);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(xr[u % 3], wr[u & 1]);
                    if (st + u + 1 >= n_stage) break;
                }
            }
        }
    } else {
        u32x4 cur[4], nxt[4];                            // the stage being multiplied and the next one, in flight
        const int lr = lane >> 3, lc = lane & 7;
        auto fetch = [&](int st, u32x4 (&r)[4]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const long long t = min(t0 + 8 * j + lr, last);          // tokens past the workgroup's re-read its last one
                r[j] = *reinterpret_cast<const u32x4*>(x + t * d + kw0 + st * KSTAGE + lc * 8);
            }
        };
        if (n_stage > 0) fetch(0, cur);
        for (int st = 0; st < n_stage; ++st) {
            if (st + 1 < n_stage) fetch(st + 1, nxt);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int row = 8 * j + lr;
                *reinterpret_cast<u32x4*>(stage + row * KSTAGE + ((lc ^ ((row >> 1) & 7)) * 8)) = cur[j];
            }
            const int ks0 = (kw0 + st * KSTAGE) / 16;
#pragma unroll
            for (int u = 0; u < KSTAGE / 16; ++u) {
                const int row = lane & 31;
                const bf16x8 a = *reinterpret_cast<const bf16x8*>(stage + row * KSTAGE + (((2 * u + (lane >> 5)) ^ ((row >> 1) & 7)) * 8));
#pragma unroll
                for (int p = 0; p < PANELS; ++p) {
                    const bf16x8 b = *reinterpret_cast<const bf16x8*>(wlane + ((size_t)(ks0 + u) * PANELS + p) * 512);
                    acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[p], 0, 0, 0);
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) cur[j] = nxt[j];
        }
    }
    {
        const long long tr = min(t0 + (lane & 31), last);
        const uint16_t* xrow = x + tr * d + 8 * (lane >> 5);
        for (int ks = (kw0 + n_stage * KSTAGE) / 16; ks < (kw0 + KSW) / 16; ++ks) {
            const bf16x8 a = *reinterpret_cast<const bf16x8*>(xrow + ks * 16);
#pragma unroll
            for (int p = 0; p < PANELS; ++p) {
                const bf16x8 b = *reinterpret_cast<const bf16x8*>(wlane + ((size_t)ks * PANELS + p) * 512);
                acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[p], 0, 0, 0);
            }
        }
    }
    __syncthreads();                                     // every wavefront is done with its staging tile: the partial sums overwrite them
    constexpr int RS = 32 * PANELS + 4;                   // row stride of the logits in LDS
    if constexpr (WAVES == 4) {
        // add the four partial sums in wavefront order
        for (int w = 0; w < 4; ++w) {
            if (wave == w && w < 3) {
#pragma unroll
                for (int p = 0; p < PANELS; ++p)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        float* slot = &red[(p * 16 + v) * 64 + lane];
                        *slot = (w == 0) ? acc[p][v] : *slot + acc[p][v];
                    }
            }
            if (w < 3) __syncthreads();
        }
        if (wave == 3) {
            // accumulator v: token 8*(v/4) + 4*(lane/32) + v%4 of this workgroup, expert panel*32 + lane%32.
            // First every partial sum is read (the logits overwrite the same LDS), then the logits are written.
#pragma unroll
            for (int p = 0; p < PANELS; ++p) {
                const int e = p * 32 + (lane & 31);
                const float b = (bias != nullptr && e < E) ? bias[e] : 0.f;
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[p][v] = red[(p * 16 + v) * 64 + lane] + acc[p][v] + b;
            }
            // (a wavefront's LDS accesses execute in program order, so these reads precede the writes below)
#pragma unroll
            for (int p = 0; p < PANELS; ++p) {
                const int e = p * 32 + (lane & 31);
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int tl = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                    red[tl * RS + e] = acc[p][v];
                    if (logits != nullptr && t0 + tl <= last && e < E) logits[(t0 + tl) * E + e] = acc[p][v];
                }
            }
        }
    } else {
        // panel by panel: all partial sums side by side; a wavefront adds those of 16 / WAVES accumulators, in wavefront order
        static_assert(16 % WAVES == 0, "whole accumulators a wavefront");
        constexpr int SHARE = 16 / WAVES;
        float sum[PANELS][SHARE];
        const auto token = [&](int i) { const int v = wave * SHARE + i; return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); };
#pragma unroll
        for (int p = 0; p < PANELS; ++p) {
            if (p > 0) __syncthreads();
#pragma unroll
            for (int v = 0; v < 16; ++v) red[(wave * 16 + v) * 64 + lane] = acc[p][v];
            __syncthreads();
            const int e = p * 32 + (lane & 31);
            const float b = (bias != nullptr && e < E) ? bias[e] : 0.f;
#pragma unroll
            for (int i = 0; i < SHARE; ++i) {
                float t = red[(wave * SHARE + i) * 64 + lane];
#pragma unroll
                for (int w = 1; w < WAVES; ++w) t += red[(w * 16 + wave * SHARE + i) * 64 + lane];
                sum[p][i] = t + b;
                if (logits != nullptr && t0 + token(i) <= last && e < E) logits[(t0 + token(i)) * E + e] = sum[p][i];
            }
        }
        __syncthreads();                                 // the sums have been read: the logits overwrite them
#pragma unroll
        for (int p = 0; p < PANELS; ++p)
#pragma unroll
            for (int i = 0; i < SHARE; ++i) red[token(i) * RS + p * 32 + (lane & 31)] = sum[p][i];
    }
    __syncthreads();
    // the gate: 8 lanes per token, 4 * PANELS logits per lane
    if (threadIdx.x >= 256) return;
    const int tl = threadIdx.x >> 3;
    const auto select = [&](auto full) {
        gate_select<8, 4 * PANELS, KMAX, false, decltype(full)::value>(red + tl * RS, true, threadIdx.x & 7, t0 + tl <= last, t0 + tl, E, k, topk_idx, topk_w);
    };
    // Whole panels select without the question which logits exist.  Asked here: 20000 tokens, d 2048, top-4, 32 experts 18.4 -> 18.1 us;
    // 65536, d 1024, top-8, 128 experts 65.4 -> 64.7, 256 experts 244.6 -> 239.7, and other numbers of experts lose nothing by the
    // second copy.  In a kernel of its own for whole panels the compiler orders the loads of x otherwise: 128 experts 77.
    if (E == 32 * PANELS) select(std::true_type());
    else select(std::false_type());
}

template <int KMAX>
__global__ __launch_bounds__(256) void router_gate_f32_kernel(const float* __restrict__ x, const float* __restrict__ w_g,
                                                              const float* __restrict__ bias, int d, int E, int k,
                                                              float* __restrict__ logits, int32_t* __restrict__ topk_idx,
                                                              float* __restrict__ topk_w) {
    __shared__ __attribute__((aligned(16))) float row[MOE_MAX_EXPERTS];
    const long long t = blockIdx.x;
    const int e = threadIdx.x;
    if (e < E) {
        float s = 0.f;
        for (int i = 0; i < d; ++i) s = fmaf(x[t * d + i], w_g[(size_t)i * E + e], s);
        s += bias ? bias[e] : 0.f;
        row[e] = s;
        if (logits != nullptr) logits[t * E + e] = s;
    }
    __syncthreads();
    gate_select<16, MOE_MAX_EXPERTS / 16, KMAX, false, false>(row, true, threadIdx.x & 15, threadIdx.x < 16, t, E, k, topk_idx, topk_w);
}

// Tokens of a workgroup with one panel of experts: as few, down to the number of experts (whose weights every workgroup
// reads), as spread the batch over 256 compute units in whole rounds: 10007 tokens are 501 workgroups of 20 (15.9 us)
// instead of 313 of 32 (17.8), of which 57 compute units have two; d 4096, 4096 tokens 256 of 16 (9.2) instead of 128 (12.8).
constexpr int kRouterUnits = 256;                // of an MI355X; on a part of one the lines lie elsewhere, the results are right
static int router_tokens(int T, int E) {
    const int rounds = (int)(((long long)T + 32 * kRouterUnits - 1) / (32 * kRouterUnits));
    const int even = (int)(((long long)T + (long long)kRouterUnits * rounds - 1) / ((long long)kRouterUnits * rounds)), least = E < 8 ? 8 : E;
    return even > least ? even : least;
}
// Wavefronts of a workgroup (measured at the kernel) and the order of the loads.  One panel of experts: sixteen for a handful of
// workgroups; then weights one and activations two stages ahead, eight wavefronts up to two workgroups a compute unit and 52 MB
// of x, then four, if the reduction is long and few lanes fetch weights; otherwise one stage ahead, sixteen wavefronts up to one
// workgroup a compute unit and 44 MB, then four.  Two panels: sixteen up to 96 workgroups, eight up to two a compute
// unit and 52 MB, otherwise sixteen up to one and then four.  Three and four: sixteen (whose weights a workgroup shares with
// itself only) up to one a compute unit, then eight, of four panels past 80 MB and up to two a compute unit four.  More
// than four panels: four, the accumulators of more do not fit.
// One stage ahead / two, 39000 random batches, times as fast by E, d: up to 16, 1025 to 2048 1.05, from there on 1.17; 24, over 2048
// 1.09; but 32 0.97, and up to 24 with d 640 to 1024 and more than 16384 tokens 0.97, d up to 512 0.92, e.g. 38892 tokens, d 256,
// E 2 8.8 us / 11.0; 9082, d 1792, E 32 12.2 / 14.6.  Between 1 and 512 tokens nothing changed; 513 to 640 gained as much as 640 to 1024.
// Two panels, sixteen (four past 8192 tokens) / eight: 3072 to 8192 tokens 1.05 up to 12 M elements, 1.01 up to 26 M, past 8192 tokens
// 1.14, 1.05, and 1.00 from 32 M on (worst 0.88 at d > 4096).  Four panels, four / eight, 8193 to 16384 tokens: 1.12 up to 40 M, 0.97 past it.
constexpr int kRouterFewTokens = 512, kRouterFewTokens2 = 3072;
constexpr long long kRouterNearElems = 26ll << 20, kRouterSmallElems = 22ll << 20, kRouterFarElems = 40ll << 20;
constexpr int kRouterAheadLimit = 1 << 25;       // d from which a panel of weights passes the 2^31 bytes that the descriptor's offsets tell apart
template <int PANELS, int WAVES, bool AHEAD = false>
static void launch_fused(const uint16_t* x, const uint16_t* packed, const float* bias, int T, int d, int E, int k, float* logits,
                         int32_t* idx, float* w, hipStream_t s) {
    const int tokens = AHEAD ? router_tokens(T, E) : 32;
    const dim3 grid((unsigned)((T + tokens - 1) / tokens)), block(64 * WAVES);
    const size_t lds = router_lds_floats(PANELS, WAVES) * sizeof(float);
    if (k <= 2) hipLaunchKernelGGL((router_gate_bf16_kernel<PANELS, 2, WAVES, AHEAD>), grid, block, lds, s, x, packed, bias, T, d, E, k, logits, idx, w, tokens);
    else if (k <= 8) hipLaunchKernelGGL((router_gate_bf16_kernel<PANELS, 8, WAVES, AHEAD>), grid, block, lds, s, x, packed, bias, T, d, E, k, logits, idx, w, tokens);
    else hipLaunchKernelGGL((router_gate_bf16_kernel<PANELS, MOE_MAX_TOPK, WAVES, AHEAD>), grid, block, lds, s, x, packed, bias, T, d, E, k, logits, idx, w, tokens);
}

int launch_router_gate(const void* x, moe_dtype_t dt, const void* packed, const float* bias, int T, int d, int E, int k,
                       float* logits, int32_t* idx, float* w, hipStream_t s) {
    LaunchTimer timer(MOE_K_ROUTER, s);
    if (dt == MOE_BF16) {
        const uint16_t* xs = (const uint16_t*)x;
        const uint16_t* ps = (const uint16_t*)packed;
        const bool round = T <= 32 * kRouterUnits, two = T <= 64 * kRouterUnits;          // at most one (two) workgroups of 32 tokens a compute unit
        const bool near = (long long)T * d <= kRouterNearElems;
        const bool ahead = d < kRouterAheadLimit && (E <= 16 ? d > 1024 : E <= 24 && d > 2048);
        const auto fused1 = T <= kRouterFewTokens ? launch_fused<1, 16>
                            : ahead ? (two && near ? launch_fused<1, 8, true> : launch_fused<1, 4, true>)
                            : round && (long long)T * d <= kRouterSmallElems ? launch_fused<1, 16> : launch_fused<1, 4>;
        const auto fused2 = T <= kRouterFewTokens2 ? launch_fused<2, 16>
                            : two && near ? launch_fused<2, 8> : round ? launch_fused<2, 16> : launch_fused<2, 4>;
        const auto fused4 = round ? launch_fused<4, 16> : two && (long long)T * d > kRouterFarElems ? launch_fused<4, 4> : launch_fused<4, 8>;
        switch (padded_experts(E) / 32) {
            case 1: fused1(xs, ps, bias, T, d, E, k, logits, idx, w, s); break;
            case 2: fused2(xs, ps, bias, T, d, E, k, logits, idx, w, s); break;
            case 3: (round ? launch_fused<3, 16> : launch_fused<3, 8>)(xs, ps, bias, T, d, E, k, logits, idx, w, s); break;
            case 4: fused4(xs, ps, bias, T, d, E, k, logits, idx, w, s); break;
            case 5: (launch_fused<5, 4>)(xs, ps, bias, T, d, E, k, logits, idx, w, s); break;
            case 6: (launch_fused<6, 4>)(xs, ps, bias, T, d, E, k, logits, idx, w, s); break;
            case 7: (launch_fused<7, 4>)(xs, ps, bias, T, d, E, k, logits, idx, w, s); break;
            default: launch_fused<8, 4>(xs, ps, bias, T, d, E, k, logits, idx, w, s); break;
        }
    } else {
        const float* xf = (const float*)x;
        const float* wf = (const float*)packed;
        if (k <= 2) hipLaunchKernelGGL(router_gate_f32_kernel<2>, dim3((unsigned)T), dim3(256), 0, s, xf, wf, bias, d, E, k, logits, idx, w);
        else if (k <= 8) hipLaunchKernelGGL(router_gate_f32_kernel<8>, dim3((unsigned)T), dim3(256), 0, s, xf, wf, bias, d, E, k, logits, idx, w);
        else hipLaunchKernelGGL(router_gate_f32_kernel<MOE_MAX_TOPK>, dim3((unsigned)T), dim3(256), 0, s, xf, wf, bias, d, E, k, logits, idx, w);
    }
    return check_launch("moe_router_gate launch");
}

}  // namespace moe
