// fp32 path of moe_expert_ffn_grouped (paper Section 2.2 / Fig. 2b, "FFN
// computations" of the resident experts) as two grouped GEMMs on the fp32
// matrix instruction (v_mfma_f32_32x32x2_f32: full fp32 products and sums, 256
// flop per clock and compute unit):
//   up  : H = silu(A W1_e) * (A W3_e)     (both products in one pass over A)
//   down: out = H W2_e
//
// Tile.  A workgroup owns 32 rows x 32 columns of outputs (of both products in
// the up projection); its four wavefronts split every 32-deep stage of the
// reduction among them, 8 k each, and add their partial sums through LDS in
// wavefront order.  At 64 cycles per matrix instruction the operands of even so
// small a tile arrive in time (12 KB per stage from L2, 3 LDS reads per two
// instructions), and it is the small tile that keeps the chip busy: ragged
// buckets waste at most 31 rows, the number of tiles divides well over 256
// compute units, and four to seven workgroups share one, so that one's barrier
// is another's turn.  Measured (2000 routes in 8 skewed buckets, d = 1024, f = 2816),
// up / down in us: 231 / 128 (100 and 90 of the 157 TFLOP/s); 64 x 64 tiles with one
// wavefront per 32 x 32 block 253 / 159, 32 x 64 tiles 243 / 145, 64-deep stages
// 286 / 146; fused multiply-adds on 64 x 64 tiles, without matrix instructions,
// 359 / 292.  Without loads and LDS writes this loop takes 189 / 101: the rest is
// the copy to LDS.
//
// Pipeline.  While stage s multiplies from registers, stage s + 1 is read from
// LDS, s + 2 is written there and the loads of s + 3 and s + 4 are in flight, one
// barrier per stage.  The inner loop computes no addresses: a stage's position
// goes into the scalar base, the lane's offset stays.
//
// Weights stay row-major as given ([W1 | W3 | W2] per expert).  A is read from
// LDS as four consecutive k per lane, so matrix instruction q of a group of four
// multiplies k = q and k = 4 + q, and B follows the same order.  Both LDS tiles
// are padded so that all accesses are conflict-free.  Every XCD takes a
// contiguous share of the tile list (expert -> column tile -> row tile), so that
// the row tiles that share a weight panel run on one L2.
#include "ffn_plan.h"

namespace moe {

typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kF32Tile = kF32TileRows;   // rows and columns of a tile
constexpr int kF32Stage = 32;        // k of one LDS stage
constexpr int kF32Waves = 4;         // wavefronts of a workgroup, each 8 k of a stage
constexpr int kF32Xcds = 8;

size_t packed_bytes_f32(int E, int d, int f) { return (size_t)E * 3 * d * f * sizeof(float); }

int launch_pack_f32(const float* w1, const float* w3, const float* w2, int E, int d, int f, float* packed, hipStream_t s) {
    // per expert: [W1 d*f | W3 d*f | W2 f*d], each matrix row-major as given
    const size_t m = (size_t)d * f * sizeof(float);
    const float* src[3] = {w1, w3, w2};
    for (int i = 0; i < 3; ++i) {
        hipError_t e = hipMemcpy2DAsync((char*)packed + i * m, 3 * m, src[i], m, m, E, hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return hip_fail(e, "moe_pack_weights copy");
    }
    return MOE_OK;
}

template <bool UP>
__global__ __launch_bounds__(256) void ffn_f32_kernel(const float* __restrict__ A, const float* __restrict__ packed,
                                                      int d, int f, float* __restrict__ C, const int32_t* __restrict__ plan) {
    constexpr int NP = UP ? 2 : 1;                                        // products
    constexpr int AST = kF32Stage + 4, BST = kF32Tile + 8;                // row strides: 16 rows of A, and rows k and k + 4 of B, fall on distinct banks
    constexpr int A_FLOATS = kF32Tile * AST, B_FLOATS = kF32Stage * BST, STAGE = A_FLOATS + NP * B_FLOATS;
    constexpr int RED = kF32Waves * NP * 16 * 64;                         // partial sums [wavefront][product][16][64]
    static_assert(kF32Tile * kF32Stage == 4 * 256, "one 16-byte piece of each operand per thread and stage");
    __shared__ __attribute__((aligned(16))) float smem[2 * STAGE > RED ? 2 * STAGE : RED];
    const int K = UP ? d : f, NC = UP ? f : d;                            // reduction length, output columns
    const int NT = (NC + kF32Tile - 1) / kF32Tile;

    // which tile: the tile list is cut into one contiguous range per XCD (workgroups go round-robin to the XCDs)
    const int32_t* prefix = plan + kPlanTiles0;
    const int n_listed = plan[0];
    const long long total = (long long)prefix[n_listed] * NT, per_xcd = (total + kF32Xcds - 1) / kF32Xcds;
    const long long slot = blockIdx.x / kF32Xcds, t = (long long)(blockIdx.x % kF32Xcds) * per_xcd + slot;
    if (slot >= per_xcd || t >= total) return;
    int lo = 0, hi = n_listed - 1;                                        // last listed bucket whose first tile is <= t
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((long long)prefix[mid] * NT <= t) lo = mid; else hi = mid - 1;
    }
    const int mt_e = prefix[lo + 1] - prefix[lo];
    const int rem = (int)(t - (long long)prefix[lo] * NT);
    const int nt = rem / mt_e, r0 = (rem - nt * mt_e) * kF32Tile;
    const int rows = min(kF32Tile, plan[kPlanCount + lo] - r0), n0 = nt * kF32Tile;
    const RowMap rm = row_map<true>(plan, lo, r0, rows);
    const bool merged = rm.merged;
    const float* We = packed + (size_t)plan[kPlanExpert + lo] * 3 * d * f;
    const float* Bbase = UP ? We : We + (size_t)2 * d * f;                // W1 (W3 follows it) or W2
    const float* Abase = merged ? A : A + (size_t)rm.row0 * K;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // A thread's piece of a stage: 4 consecutive k of a row of A, 4 columns of a k row of B.  Rows and columns past the
    // tile's end re-read its last ones (their outputs are never stored).  The last stage of a reduction that is no
    // multiple of 32 reads the last 32 k and counts those that came before it as zero; a reduction shorter than 32
    // re-reads its last k and counts that as zero.
    const int ar = tid / 8, ak = (tid % 8) * 4, bk = tid / 8, bc = (tid % 8) * 4;
    const int arow = min(ar, rows - 1);
    const uint32_t a_off = (uint32_t)(merged ? buffer_row(rm, arow) : arow) * (uint32_t)K + (uint32_t)min(ak, K - 4);
    const uint32_t b_off = (uint32_t)min(bk, K - 1) * (uint32_t)NC + (uint32_t)min(n0 + bc, NC - 4);
    const int k_last = max(K - kF32Stage, 0);
    struct Regs { float4 a, b[NP]; };
    auto fetch = [&](int s, Regs& r) {
        const int k0 = min(s * kF32Stage, k_last);
        r.a = *reinterpret_cast<const float4*>(Abase + k0 + a_off);
#pragma unroll
        for (int p = 0; p < NP; ++p) r.b[p] = *reinterpret_cast<const float4*>(Bbase + (size_t)p * d * f + (size_t)k0 * NC + b_off);
    };
    auto keep = [](const float4& v, bool in) { return make_float4(in ? v.x : 0.f, in ? v.y : 0.f, in ? v.z : 0.f, in ? v.w : 0.f); };
    auto stage = [&](int s, Regs& r, float* buf) {
        if ((s + 1) * kF32Stage > K) {                                    // wave-uniform: the ragged last stage only
            const int k0 = min(s * kF32Stage, k_last), lo_k = s * kF32Stage - k0;
            r.a = keep(r.a, ak >= lo_k && k0 + ak < K);
#pragma unroll
            for (int p = 0; p < NP; ++p) r.b[p] = keep(r.b[p], bk >= lo_k && k0 + bk < K);
        }
        *reinterpret_cast<float4*>(buf + ar * AST + ak) = r.a;
#pragma unroll
        for (int p = 0; p < NP; ++p) *reinterpret_cast<float4*>(buf + A_FLOATS + p * B_FLOATS + bk * BST + bc) = r.b[p];
    };
    // this wavefront's operands of a stage: lane l holds row (column) l % 32 and the four k from 8 * wave + 4 * (l / 32)
    struct Frags { float4 a; float b[NP][4]; };
    const float* as = smem + (lane & 31) * AST + 8 * wave + 4 * (lane >> 5);
    const float* bs = smem + A_FLOATS + (8 * wave + 4 * (lane >> 5)) * BST + (lane & 31);
    auto read = [&](int buf, Frags& fr) {
        fr.a = *reinterpret_cast<const float4*>(as + buf * STAGE);
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) fr.b[p][q] = bs[buf * STAGE + p * B_FLOATS + q * BST];
    };
    f32x16 acc[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[p][v] = 0.f;
    auto multiply = [&](const Frags& fr) {
        const float av[4] = {fr.a.x, fr.a.y, fr.a.z, fr.a.w};
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int p = 0; p < NP; ++p) acc[p] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[q], fr.b[p][q], acc[p], 0, 0, 0);
    };

    const int n_stage = (K + kF32Stage - 1) / kF32Stage;                  // stages past the end are fetched and staged, never multiplied
    Regs even, odd;
    Frags f0, f1;
    fetch(0, even);
    fetch(1, odd);
    stage(0, even, smem);
    fetch(2, even);
    __syncthreads();
    read(0, f0);
    stage(1, odd, smem + STAGE);
    fetch(3, odd);
    __syncthreads();
    for (int s = 0; s + 1 < n_stage; s += 2) {
        read(1, f1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(f0);
        stage(s + 2, even, smem);                                         // its previous contents were read before the last barrier
        fetch(s + 4, even);
        __syncthreads();
        read(0, f0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(f1);
        stage(s + 3, odd, smem + STAGE);
        fetch(s + 5, odd);
        __syncthreads();
    }
    if (n_stage & 1) multiply(f0);

    // add the four partial sums in wavefront order; a wavefront finishes 4 of the 16 accumulator rows
    __syncthreads();                                                      // the stages have been read by everyone
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int v = 0; v < 16; ++v) smem[((wave * NP + p) * 16 + v) * 64 + lane] = acc[p][v];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int v = wave * 4 + i;
        float sum[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            sum[p] = smem[(p * 16 + v) * 64 + lane];
#pragma unroll
            for (int w = 1; w < kF32Waves; ++w) sum[p] += smem[((w * NP + p) * 16 + v) * 64 + lane];
        }
        // accumulator v: row 8 * (v / 4) + 4 * (lane / 32) + v % 4, column lane % 32
        const int r = 8 * wave + 4 * (lane >> 5) + i, c = n0 + (lane & 31);
        const float u = sum[0];
        const size_t at = buffer_row(rm, min(r, rows - 1));
        if (r < rows && c < NC) C[at * NC + c] = UP ? u / (1.0f + expf(-u)) * sum[NP - 1] : u;
    }
}

int launch_ffn_f32(const float* a, int N, int d, int f, int E, const float* packed, const int32_t* counts,
                   const int32_t* starts, const int32_t* placement, int local_gpu, const int32_t* group_expert,
                   int n_weights, float* out, int32_t* plan, bool plan_ready, float* H, hipStream_t s) {
    int rc;
    if (!plan_ready) {
        PlanShape shape;
        if ((rc = ffn_plan_shape(MOE_F32, N, d, f, E, false, &shape)) != MOE_OK) return rc;
        // groups that may share an expert are merged; the row offsets of a merged bucket must fit 32 bits
        const bool mergeable = group_expert != nullptr && (size_t)N * (d > f ? d : f) < ((size_t)1 << 32);
        rc = launch_ffn_plan(counts, starts, placement, local_gpu, group_expert, n_weights, E, N, shape, mergeable, {}, plan, s);
        if (rc != MOE_OK) return rc;
    }
    const long long mt_max = (N + kF32Tile - 1) / kF32Tile + (E < N ? E : N);     // sum of ceil(n_e / 32) never exceeds this
    auto grid_for = [&](int columns) { return (mt_max * ((columns + kF32Tile - 1) / kF32Tile) + kF32Xcds - 1) / kF32Xcds * kF32Xcds; };
    if (grid_for(f) > 0x7FFFFFFFll || grid_for(d) > 0x7FFFFFFFll)
        return fail(MOE_ERR_UNSUPPORTED, "moe_expert_ffn_grouped: too many tiles for one launch");
    {
        LaunchTimer timer(MOE_K_FFN_UP, s);
        hipLaunchKernelGGL(ffn_f32_kernel<true>, dim3((unsigned)grid_for(f)), dim3(256), 0, s, a, packed, d, f, H, plan);
        if ((rc = check_launch("moe_expert_ffn_grouped up launch")) != MOE_OK) return rc;
    }
    {
        LaunchTimer timer(MOE_K_FFN_DOWN, s);
        hipLaunchKernelGGL(ffn_f32_kernel<false>, dim3((unsigned)grid_for(d)), dim3(256), 0, s, (const float*)H, packed, d, f, out, plan);
        if ((rc = check_launch("moe_expert_ffn_grouped down launch")) != MOE_OK) return rc;
    }
    return MOE_OK;
}

}  // namespace moe
