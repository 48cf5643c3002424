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
// small a tile arrive in time (12 KB per stage from L2, one 16-byte LDS read per eight
// instructions in the up projection, per four in the down), and it is the small tile that
// keeps the chip busy: ragged buckets waste at most 31 rows, the number of tiles divides well over 256
// compute units, and four workgroups (up) or seven (down) share one, so that one's barrier
// is another's turn.  Measured when both operands went through LDS (2000 routes in 8 skewed buckets, d = 1024,
// f = 2816), up / down in us: 231 / 128 (100 and 90 of the 157 TFLOP/s); 64 x 64 tiles with one
// wavefront per 32 x 32 block 253 / 159, 32 x 64 tiles 243 / 145, 64-deep stages
// 286 / 146; fused multiply-adds on 64 x 64 tiles, without matrix instructions,
// 359 / 292.  Without loads and LDS writes that loop took 189 / 101: the rest was
// the copy to LDS, of which only A's is left.
//
// Weights.  The four k of a column lie side by side ([K / 4][columns][4] per matrix,
// [W1 | W3 | W2] per expert), so that the 16 bytes that a thread fetches of a stage
// are what its lane multiplies: B goes straight into registers, four stages ahead, a
// wavefront reading 512 contiguous bytes of two such rows.  A goes through LDS
// because a wavefront's 8 k of 32 rows are 32 bytes a row: fetched by the lanes that
// multiply them, without LDS, layers took 1.0 to 1.65 times as long.  Both
// operands through LDS, B row-major: 1064 tokens, top-2, d 500, f 400, 4 experts, up 30.5
// us and down 18.5, now 27.4 and 17.0; 116 routes of one expert, f 2048, down 15.7, now 14.9, up
// by its one to eight stages (d 32 to 256) 5.3 to 8.5, now 5.4 to 8.0, five (d 152) 7.25, now 7.1.
//
// Pipeline.  While stage s multiplies, the A of stage s + 1 is read from LDS, that of
// s + 2 is written there and the loads of s + 3 and s + 4 are in flight, one
// barrier per stage.  The inner loop computes no addresses: a stage's position
// goes into the scalar base, the lane's offset stays.
//
// A is read from LDS as four consecutive k per lane, so matrix instruction q of a group of four
// multiplies k = q and k = 4 + q, and B follows the same order.  The LDS tile
// is padded so that all accesses are conflict-free.  Every XCD takes a
// contiguous share of the tile list (expert -> column tile -> row tile), so that
// the row tiles that share a weight panel run on one L2.
//
// Large batches take the bf16 matrix instruction on values split in three, see further down.
#include "ffn_plan.h"

namespace moe {

typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kF32Tile = kF32TileRows;   // rows and columns of a tile
constexpr int kF32Stage = 32;        // k of one LDS stage
constexpr int kF32Waves = 4;         // wavefronts of a workgroup, each 8 k of a stage
constexpr int kF32Xcds = 8;

size_t packed_bytes_f32(int E, int d, int f) { return (size_t)E * 3 * d * f * sizeof(float); }

// per expert [W1 d*f | W3 d*f | W2 f*d]; a matrix of K rows and NC columns as [K / 4][NC][4]: the four k of a column side by side.
// One thread per 16 bytes, blockIdx.y = matrix; a matrix of 2^30 units and more takes a loop over them, as HIP launches fewer than 2^32
// threads along a dimension of the grid.
__global__ __launch_bounds__(256) void pack_f32_kernel(const float* __restrict__ w1, const float* __restrict__ w3, const float* __restrict__ w2,
                                                       int d, int f, long long units, float4* __restrict__ packed) {
    const int e = blockIdx.y / 3, which = blockIdx.y - 3 * e, NC = which == 2 ? d : f;
    const float* src = (which == 0 ? w1 : (which == 1 ? w3 : w2)) + e * units * 4;
    float4* out = packed + blockIdx.y * units;
    for (long long r = (long long)blockIdx.x * 256 + threadIdx.x; r < units; r += (long long)gridDim.x * 256) {
        const long long q = r >> 32 ? r / NC : (uint32_t)r / (uint32_t)NC;
        const float* s = src + q * 4 * NC + (r - q * NC);
        out[r] = make_float4(s[0], s[NC], s[2 * (size_t)NC], s[3 * (size_t)NC]);
    }
}

int launch_pack_f32(const float* w1, const float* w3, const float* w2, int E, int d, int f, float* packed, hipStream_t s) {
    const long long units = (long long)d * f / 4;
    const unsigned grid = (unsigned)(units < (1ll << 30) ? (units + 255) / 256 : 1 << 22);
    hipLaunchKernelGGL(pack_f32_kernel, dim3(grid, 3 * E), dim3(256), 0, s, w1, w3, w2, d, f, units, (float4*)packed);
    return check_launch("moe_pack_weights launch");
}

template <bool UP>
__global__ __launch_bounds__(256) void ffn_f32_kernel(const float* __restrict__ A, const float* __restrict__ packed,
                                                      int d, int f, float* __restrict__ C, const int32_t* __restrict__ plan) {
    constexpr int NP = UP ? 2 : 1;                                        // products
    constexpr int AST = kF32Stage + 4, STAGE = kF32Tile * AST;            // row stride: 16 rows of A fall on distinct banks
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

    // A thread's piece of a stage: four consecutive k of a row of A and of a column of B.  The latter is what its lane multiplies:
    // lane l of wavefront w holds the k from 8 w + 4 (l / 32) of row (column) l % 32.  Rows and columns past the
    // tile's end re-read its last ones (their outputs are never stored).  The last stage of a reduction that is no
    // multiple of 32 reads the last 32 k and counts those that came before it as zero; a reduction shorter than 32
    // re-reads its last k and counts that as zero.
    const int ar = tid / 8, ak = (tid % 8) * 4, bk = (tid / 32) * 4, bc = tid % 32;
    const int arow = min(ar, rows - 1);
    const uint32_t a_off = (uint32_t)(merged ? buffer_row(rm, arow) : arow) * (uint32_t)K + (uint32_t)min(ak, K - 4);
    const uint32_t b_off = (uint32_t)min(bk, K - 4) * (uint32_t)NC + 4u * (uint32_t)min(n0 + bc, NC - 1);
    const int k_last = max(K - kF32Stage, 0);
    struct Regs { float4 a, b[NP]; };
    auto fetch = [&](int s, Regs& r) {
        const int k0 = min(s * kF32Stage, k_last);
        r.a = *reinterpret_cast<const float4*>(Abase + k0 + a_off);
#pragma unroll
        for (int p = 0; p < NP; ++p) r.b[p] = *reinterpret_cast<const float4*>(Bbase + (size_t)p * d * f + (size_t)k0 * NC + b_off);
    };
    // what counts of stage s: all, but in the ragged last one
    auto keep = [&](int s, int k, float4& v) {
        if ((s + 1) * kF32Stage <= K) return;                             // wave-uniform
        const int k0 = min(s * kF32Stage, k_last);
        const bool in = k >= s * kF32Stage - k0 && k0 + k < K;
        v = make_float4(in ? v.x : 0.f, in ? v.y : 0.f, in ? v.z : 0.f, in ? v.w : 0.f);
    };
    auto stage = [&](int s, Regs& r, int buf, auto whole) {
        if (!decltype(whole)::value) keep(s, ak, r.a);
        *reinterpret_cast<float4*>(smem + buf * STAGE + ar * AST + ak) = r.a;
    };
    const float* as = smem + (lane & 31) * AST + 8 * wave + 4 * (lane >> 5);
    auto read = [&](int buf) { return *reinterpret_cast<const float4*>(as + buf * STAGE); };
    f32x16 acc[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[p][v] = 0.f;
    auto multiply = [&](int s, const float4& a, Regs& r, auto whole) {
        if (!decltype(whole)::value)
#pragma unroll
            for (int p = 0; p < NP; ++p) keep(s, bk, r.b[p]);
        const float av[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const float bv[4] = {r.b[p].x, r.b[p].y, r.b[p].z, r.b[p].w};
                acc[p] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[q], bv[q], acc[p], 0, 0, 0);
            }
    };

    const int n_stage = (K + kF32Stage - 1) / kF32Stage;                  // stages past the end are fetched and staged, never multiplied
    Regs r[4];
    float4 fa[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        fetch(i, r[i]);
        __builtin_amdgcn_sched_barrier(0);
    }
    const std::true_type whole;
    const std::false_type ragged;
    stage(0, r[0], 0, ragged);
    __syncthreads();
    fa[0] = read(0);
    stage(1, r[1], 1, ragged);
    __syncthreads();
    auto step = [&](int s, int i, auto kind) {
        fa[(i + 1) & 1] = read((i + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(s + i, fa[i & 1], r[i], kind);
        stage(s + i + 2, r[(i + 2) & 3], i & 1, kind);                    // its previous contents were read before the last barrier
        if (decltype(kind)::value || s + i + 4 < n_stage) fetch(s + i + 4, r[i]);
        __syncthreads();
    };
    int s = 0;
    for (; (s + 6) * kF32Stage <= K; s += 4)
#pragma unroll
        for (int i = 0; i < 4; ++i) step(s, i, whole);
    for (; s < n_stage; s += 4)                                           // the last ones
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (s + i >= n_stage) break;
            step(s, i, ragged);
        }

    // add the four partial sums in wavefront order; a wavefront finishes 4 of the 16 accumulator rows.  They overwrite the stages, which
    // everyone had read before the barrier that ends the last step; there is one, a reduction has at least one stage.
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

// ---- large batches: the same products on the bf16 matrix instruction -------------------------------------------------
// An fp32 value from 2^-110 on is the sum of three bf16 values exactly (the value rounded, the remainder rounded, the rest;
// below that the last bit lies under 2^-133, the smallest bf16 value), and the
// bf16 instruction has sixteen times the fp32 one's rate: the six largest of the nine products of pieces, which leave out
// 2^-24 of a product at most, come to 2.7 times it (Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial Intelligence
// Datatype For Higher-Precision Computations", 2019, has the method).  The instruction does not round its sums to nearest, so that a
// chain of all of them is worse than fp32 (1.10e-6 of the result's norm where the fp32 kernel has 6.4e-7); a stage of 32 k
// is therefore summed from zero, smallest products first, and added with a vector addition: 2.6e-7, the largest error
// of an element 2.3e-6 against 4.7e-6 (d 1024, f 2816, 2000 routes; smaller in the same way at all sizes measured).
//
// A workgroup owns 64 rows x 64 columns of outputs, a wavefront 16 columns of it (of both products in the up
// projection).  B goes from memory into the lanes that multiply it, 8 k of a column each, and is split there; A is
// needed by all four wavefronts, so each splits 16 rows and hands the pieces on through LDS in operand order.
// Between the products of a stage the next one is split, and the one after is in flight, one barrier per stage; the
// compiler would move the loads down to their use, and all products behind all of the split, hence the scheduling barriers.  Blocks of 16 rows past the bucket's
// end are not multiplied.
//
// Bound by power for the up projection (the clock falls to 1.9 to 2.1 GHz) and by the loads and vector work of the narrower
// tile for the down projection.  2000 routes in 8 skewed buckets, d 1024, f 2816, layer 369 us on the fp32 kernel; here, one change after
// the other on one GPU: weights row-major, sixteen of a stage's eighteen loads four bytes wide, 301; the four k of a column side by side 287;
// ragged tiles last (split_tile) 279; the split of a stage between the products of the one before (stage) 270.  First against last on
// two other GPUs: 303 and 272, 309 and 279.
// The look at every operand (split_pair) is one instruction a pair; as a minimum of their magnitudes, three a pair, it made 302 315.  Also
// lost, with row-major weights and the last four without that look (293 us, 4096 routes 501): B by buffer loads with the row in a scalar
// offset, 193 -> 202 us in the up projection; the remainders by v_dot2_f32_bf16, exact and a sixth fewer vector instructions,
// 327 -> 341; both products staged through LDS 345; tiles of 128 rows 309, 512; 128 columns in the down projection 305, 515; one
// stage in flight and four wavefronts a SIMD 291, 497, but 512 routes 174 for 147.  Four stages of values under way where a tile has one
// block of rows: nothing gained (25 us a tile), and the registers cost the other tiles a workgroup a compute unit.
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kSplitBlocks = kF32SplitRows / 16;     // 16-row blocks of a tile
constexpr int kSplitStage = 32;                      // k of a stage
constexpr int kSplitCols = 64;                       // output columns of a tile
static_assert(kSplitBlocks == kF32Waves, "a wavefront splits one block of A");

// Whether the batch is large enough, every row being in a resident bucket: enough work, enough rows a bucket to fill a tile,
// and enough tiles in the smaller of the two launches to give most compute units two of these workgroups (they hide
// the loads behind each other's products; the fp32 kernel's tiles are a quarter the size).  Measured on 4800 random layers of
// 0.5e9 to 30e9 with 1 to 64 experts, uniform to skewed: inside the rule 1339, 0.995 to 1.6 times as fast, 1.27 on average.  With
// N d f >= 1.6e9 and 64 rows a bucket alone, 381 of 2855 were more than 5 % slower: 64 rows, one expert, d 4096, f 8192 166 us ->
// 297 (64 workgroups in the down projection), 512 rows, 8 experts, d 2048, f 1600 143 -> 169, 1024, d 1024, f 2048 154 -> 162; with
// 400 tiles and 1.6e9 the worst is 4874 rows, 64 experts, d 332, f 992, 0.94 times as fast.
static bool split_pays(int N, int d, int f, int E) {
    const long long tiles = (long long)(N / kF32SplitRows) * (((d < f ? d : f) + kSplitCols - 1) / kSplitCols);
    return (double)N * d * f >= 2.5e9 && N >= (long long)kF32SplitRows * E && tiles >= 400;
}

// 8 fp32 values -> their three bf16 pieces.  What is left of a value for the third piece has bits below that piece's last one
// exactly if the three do not add up to the value (a magnitude below 2^-110 whose last bit lies under 2^-133): lost collects them.
__device__ __forceinline__ void split_pair(float a, float b, u32x4 (&piece)[3], int i, uint32_t& lost) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const f32x2 pair = {a, b};
        const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(pair, bf16x2));
        piece[p][i] = h;
        a -= __uint_as_float(h << 16);
        b -= __uint_as_float(h & 0xFFFF0000u);
    }
    piece[2][i] = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);     // the upper halves
    lost |= __float_as_uint(a) | __float_as_uint(b);
}
__device__ __forceinline__ void split_eight(const float (&v)[8], u32x4 (&piece)[3], uint32_t& lost) {
#pragma unroll
    for (int i = 0; i < 4; ++i) split_pair(v[2 * i], v[2 * i + 1], piece, i, lost);
}
constexpr uint32_t kSplitLost = 0xFFFFu;

// Which tile a workgroup owns: listed bucket, first row in it, column tile.  Every XCD first walks its contiguous share of the
// full row tiles (bucket -> column tile -> row tile: those that share a weight panel run on one L2), then the buckets' last,
// ragged ones, those of more 16-row blocks first, of which every XCD has the same mix.  The short ones run last because two or
// three workgroups share a compute unit: one more full tile at the end keeps its compute unit busy for half as long again as the others.
// Called by whole wavefronts, a lane per bucket.
__device__ __forceinline__ bool split_tile(const int32_t* __restrict__ plan, int NT, int& bucket, int& r0, int& nt) {
    const int n_listed = plan[0], lane = threadIdx.x & 63, x = blockIdx.x % kF32Xcds;
    const long long slot = blockIdx.x / kF32Xcds;
    const auto rows_of = [&](int i) { return i < n_listed ? plan[kPlanCount + i] : 0; };
    const int rows0 = rows_of(lane);                                      // the first 64 buckets, mostly all there are
    const auto rows_at = [&](int c) { return c == 0 ? rows0 : rows_of(c + lane); };
    int ragged = 0;
    for (int c = 0; c < n_listed; c += 64) ragged += __builtin_popcountll(__ballot(rows_at(c) % kF32SplitRows != 0));
    const long long full = (long long)(plan[2] - ragged) * NT, per_xcd = (full + kF32Xcds - 1) / kF32Xcds, first = x * per_xcd;
    const long long here = first >= full ? 0 : (full - first < per_xcd ? full - first : per_xcd);
    if (slot < here) {
        const long long t = first + slot;
        int before = 0;                                                   // full row tiles of the buckets already passed
        for (int c = 0; c < n_listed; c += 64) {
            const int mine = rows_at(c) / kF32SplitRows;
            int sum = mine;
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) {
                const int o = __shfl_up(sum, m, 64);
                sum += lane >= m ? o : 0;
            }
            const int i = __builtin_popcountll(__ballot((long long)(before + sum) * NT <= t));
            if (i < 64) {
                const int tiles = __builtin_amdgcn_readlane(mine, i), start = before + __builtin_amdgcn_readlane(sum, i) - tiles;
                const int rem = (int)(t - (long long)start * NT);
                bucket = c + i;
                nt = rem / tiles;
                r0 = (rem - nt * tiles) * kF32SplitRows;
                return true;
            }
            before += __builtin_amdgcn_readlane(sum, 63);
        }
        return false;
    }
    const long long t = (slot - here) * kF32Xcds + x;
    if (t >= (long long)ragged * NT) return false;
    int rank = (int)(t / NT);
    nt = (int)(t - (long long)rank * NT);
    for (int blocks = kSplitBlocks; blocks > 0; --blocks)
        for (int c = 0; c < n_listed; c += 64) {
            const int rows = rows_at(c), over = rows % kF32SplitRows;
            unsigned long long of_size = __ballot((over + 15) / 16 == blocks && over != 0);
            const int count = __builtin_popcountll(of_size);
            if (rank >= count) {
                rank -= count;
                continue;
            }
            for (; rank > 0; --rank) of_size &= of_size - 1;
            const int i = __builtin_ctzll(of_size);
            bucket = c + i;
            r0 = __builtin_amdgcn_readlane(rows - over, i);
            return true;
        }
    return false;
}

template <bool UP>
__global__ __launch_bounds__(256, 2) void ffn_f32_split_kernel(const float* __restrict__ A, const float* __restrict__ packed,
                                                               int d, int f, float* __restrict__ C, const int32_t* __restrict__ plan) {
    constexpr int NP = UP ? 2 : 1, A_UNITS = 3 * kSplitBlocks * 64;       // products; 16-byte units of A's pieces in a stage
    __shared__ u32x4 smem[2 * A_UNITS];
    const int K = UP ? d : f, NC = UP ? f : d;
    const int NT = (NC + kSplitCols - 1) / kSplitCols;

    int lo, r0, nt;
    if (!split_tile(plan, NT, lo, r0, nt)) return;
    const int rows = min(kF32SplitRows, plan[kPlanCount + lo] - r0), n0 = nt * kSplitCols;
    const RowMap rm = row_map<true>(plan, lo, r0, rows);
    const bool merged = rm.merged;
    const float* We = packed + (size_t)plan[kPlanExpert + lo] * 3 * d * f;
    const float* Bbase = UP ? We : We + (size_t)2 * d * f;
    const float* Abase = merged ? A : A + (size_t)rm.row0 * K;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // an operand of the instruction: lane l holds row (column) l % 16 and the 8 k from 8 * (l / 16).  Rows and columns past
    // the tile's end re-read its last ones (their outputs are never stored)
    const int kg = 8 * (lane >> 4), col = n0 + 16 * wave + (lane & 15), arow = min(16 * wave + (lane & 15), rows - 1);
    const uint32_t a_off = (uint32_t)(merged ? buffer_row(rm, arow) : arow) * (uint32_t)K + (uint32_t)kg;
    const uint32_t b_col = (uint32_t)min(col, NC - 1);
    const uint32_t b_off = (uint32_t)kg * (uint32_t)NC + 4u * b_col;
    const int n_full = K / kSplitStage, n_stage = (K + kSplitStage - 1) / kSplitStage;
    struct Raw { float a[8], b[NP][8]; };
    auto fetch = [&](int s, Raw& r) {                                     // a whole stage
        const int k0 = s * kSplitStage;
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int h = 0; h < 8; h += 4) {
                const float4 q = *reinterpret_cast<const float4*>(Bbase + (size_t)p * d * f + (size_t)(k0 + h) * NC + b_off);
                r.b[p][h] = q.x; r.b[p][h + 1] = q.y; r.b[p][h + 2] = q.z; r.b[p][h + 3] = q.w;
            }
#pragma unroll
        for (int h = 0; h < 8; h += 4) {
            const float4 q = *reinterpret_cast<const float4*>(Abase + k0 + (a_off + h));
            r.a[h] = q.x; r.a[h + 1] = q.y; r.a[h + 2] = q.z; r.a[h + 3] = q.w;
        }
    };
    auto fetch_last = [&](int s, Raw& r) {                                // the one that the reduction ends in: k past the end count as zero
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int h = 0; h < 8; h += 4) {
                const int k = s * kSplitStage + kg + h;
                const float4 q = *reinterpret_cast<const float4*>(Bbase + (size_t)p * d * f + (size_t)min(k, K - 4) * NC + 4u * b_col);
                const bool in = k < K;
                r.b[p][h] = in ? q.x : 0.f; r.b[p][h + 1] = in ? q.y : 0.f; r.b[p][h + 2] = in ? q.z : 0.f; r.b[p][h + 3] = in ? q.w : 0.f;
            }
#pragma unroll
        for (int h = 0; h < 8; h += 4) {
            const int k = s * kSplitStage + kg + h;
            const float4 q = *reinterpret_cast<const float4*>(Abase + (a_off - kg + min(k, K - 4)));
            const bool in = k < K;
            r.a[h] = in ? q.x : 0.f; r.a[h + 1] = in ? q.y : 0.f; r.a[h + 2] = in ? q.z : 0.f; r.a[h + 3] = in ? q.w : 0.f;
        }
    };
    struct Frags { u32x4 b[NP][3]; };
    uint32_t a_lost = 0, b_lost = 0;                                      // of this lane's row of A and column of B
    auto convert = [&](const Raw& r, Frags& fr, int buf) {
        u32x4 pa[3];
        split_eight(r.a, pa, a_lost);
#pragma unroll
        for (int q = 0; q < 3; ++q) smem[buf * A_UNITS + (q * kSplitBlocks + wave) * 64 + lane] = pa[q];
#pragma unroll
        for (int p = 0; p < NP; ++p) split_eight(r.b[p], fr.b[p], b_lost);
    };

    f32x4 acc[kSplitBlocks][NP];
#pragma unroll
    for (int m = 0; m < kSplitBlocks; ++m)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[m][p][v] = 0.f;
    auto loop = [&](auto active) {
        constexpr int NA = decltype(active)::value;                       // row blocks that hold rows of the bucket
        constexpr int MG = NA < 4 / NP ? NA : 4 / NP;                     // row blocks at a time: up to four chains of matrix instructions
        auto multiply = [&](const Frags& fr, int buf) {
#pragma unroll
            for (int m0 = 0; m0 < NA; m0 += MG) {
                u32x4 a[MG][3];
                f32x4 sum[MG][NP];
#pragma unroll
                for (int m = 0; m < MG; ++m)
#pragma unroll
                    for (int q = 0; q < 3; ++q) a[m][q] = smem[buf * A_UNITS + (q * kSplitBlocks + min(m0 + m, NA - 1)) * 64 + lane];
                constexpr int piece_a[6] = {2, 0, 1, 1, 0, 0}, piece_b[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
                for (int q = 0; q < 6; ++q)
#pragma unroll
                    for (int m = 0; m < MG; ++m)
#pragma unroll
                        for (int p = 0; p < NP; ++p)
                            if (m0 + m < NA)
                                sum[m][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[m][piece_a[q]]),
                                                                                    __builtin_bit_cast(bf16x8, fr.b[p][piece_b[q]]),
                                                                                    q == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sum[m][p], 0, 0, 0);
#pragma unroll
                for (int m = 0; m < MG; ++m)
#pragma unroll
                    for (int p = 0; p < NP; ++p)
                        if (m0 + m < NA)
#pragma unroll
                            for (int v = 0; v < 4; ++v) acc[m0 + m][p][v] += sum[m][p][v];
            }
        };
        // The products of one stage, and between them the split of the next: a matrix instruction keeps the matrix pipe busy for 16
        // cycles, in which the wavefront issues three or four vector instructions.
        auto stage = [&](const Frags& fr, int buf, const Raw& raw, Frags& next, int next_buf) {
            constexpr int H = (NA + MG - 1) / MG, G = 6 * H, U = 4 + 4 * NP;       // groups of row blocks; of matrix instructions; pairs of values to split
            constexpr int piece_a[6] = {2, 0, 1, 1, 0, 0}, piece_b[6] = {0, 2, 1, 0, 1, 0};
            u32x4 a[2][MG][3], pa[3];
            f32x4 sum[2][MG][NP];
            auto read = [&](int h) {
#pragma unroll
                for (int m = 0; m < MG; ++m)
#pragma unroll
                    for (int q = 0; q < 3; ++q) a[h & 1][m][q] = smem[buf * A_UNITS + (q * kSplitBlocks + min(h * MG + m, NA - 1)) * 64 + lane];
            };
            auto add = [&](int h, int m, int p) {
                if (h * MG + m < NA)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[h * MG + m][p][v] += sum[h & 1][m][p][v];
            };
            read(0);
#pragma unroll
            for (int h = 0; h < H; ++h) {
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    const int g = 6 * h + q;
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int m = 0; m < MG; ++m)
#pragma unroll
                        for (int p = 0; p < NP; ++p)
                            if (h * MG + m < NA)
                                sum[h & 1][m][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[h & 1][m][piece_a[q]]),
                                                                                           __builtin_bit_cast(bf16x8, fr.b[p][piece_b[q]]),
                                                                                           q == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sum[h & 1][m][p], 0, 0, 0);
                    if (q == 1 && h + 1 < H) read(h + 1);
#pragma unroll
                    for (int u = g * U / G; u < (g + 1) * U / G; ++u) {
                        if (u < 4) split_pair(raw.a[2 * u], raw.a[2 * u + 1], pa, u, a_lost);
                        else split_pair(raw.b[(u - 4) / 4][2 * (u % 4)], raw.b[(u - 4) / 4][2 * (u % 4) + 1], next.b[(u - 4) / 4], u % 4, b_lost);
                        if (u == 3)
#pragma unroll
                            for (int i = 0; i < 3; ++i) smem[next_buf * A_UNITS + (i * kSplitBlocks + wave) * 64 + lane] = pa[i];
                    }
                    if (h > 0 && q < MG * NP) add(h - 1, q / NP, q % NP);
#pragma unroll
                    for (int i = 0; i < MG * NP; ++i) {
                        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                        if (UP && h == 0) __builtin_amdgcn_sched_group_barrier(0x2, 3, 0);
                        else __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < MG; ++m)
#pragma unroll
                for (int p = 0; p < NP; ++p) add(H - 1, m, p);
        };
        Raw even, odd;
        Frags f0, f1;
        auto get = [&](int s, Raw& r) { if (s < n_full) fetch(s, r); else if (s < n_stage) fetch_last(s, r); };
        get(0, even);
        get(1, odd);
        convert(even, f0, 0);
        __syncthreads();
        int s = 0;
        for (; s + 3 < n_full; s += 2) {
            fetch(s + 2, even);
            __builtin_amdgcn_sched_barrier(0);
            stage(f0, 0, odd, f1, 1);                                     // its LDS was read before the last barrier
            __syncthreads();
            fetch(s + 3, odd);
            __builtin_amdgcn_sched_barrier(0);
            stage(f1, 1, even, f0, 0);
            __syncthreads();
        }
        // Keeps the sums' additions in the block of the products that they read: moved into the block after the branch, two
        // of them came too early after the last matrix instruction, which the compiler does not see on every path.  The loop above
        // is one block, and its sums are needed on both ways out of it: there is nowhere to move them (held there too: up
        // to 1 % slower).
        auto settle = [&]() {
#pragma unroll
            for (int m = 0; m < NA; ++m)
#pragma unroll
                for (int p = 0; p < NP; ++p) asm volatile("" : "+v"(acc[m][p]));
        };
        for (;; s += 2) {                                                 // up to four stages, the ragged one among them
            get(s + 2, even);
            if (s + 1 < n_stage) convert(odd, f1, 1);
            multiply(f0, 0);
            settle();
            if (s + 1 >= n_stage) break;
            __syncthreads();
            get(s + 3, odd);
            if (s + 2 < n_stage) convert(even, f0, 0);
            multiply(f1, 1);
            settle();
            if (s + 2 >= n_stage) break;
            __syncthreads();
        }
    };
    const int blocks = (rows + 15) / 16;                                  // the same for all wavefronts
    switch (blocks) {
        case 1: loop(std::integral_constant<int, 1>()); break;
        case 2: loop(std::integral_constant<int, 2>()); break;
        case 3: loop(std::integral_constant<int, 3>()); break;
        default: loop(std::integral_constant<int, 4>()); break;
    }

    // which rows and columns have an operand without three exact pieces: every wavefront knows its columns and a quarter of the rows
    const auto of_16 = [](bool v) {                                       // bit i: any of lanes i, 16 + i, 32 + i, 48 + i
        const unsigned long long b = __ballot(v);
        const uint32_t h = (uint32_t)(b | b >> 32);
        return (h | h >> 16) & 0xFFFFu;
    };
    uint32_t* small = reinterpret_cast<uint32_t*>(smem);
    const uint32_t my_rows = of_16((a_lost & kSplitLost) != 0), my_cols = of_16((b_lost & kSplitLost) != 0);
    __syncthreads();                                                      // the pieces have been read by everyone
    small[wave] = my_rows;
    __syncthreads();

    // accumulator v of block m: row 16 m + 4 (lane / 16) + v, column lane % 16
    // (a sum near the smallest fp32 value has lost more bits than in plain fp32, too)
    constexpr float kMax = 3.4028234e38f, kMin = 7.7e-34f;                // the second: 2^-110
    const auto in_range = [](float v) { return fabsf(v) <= kMax && (fabsf(v) >= kMin || v == 0.f); };
    const bool small_col = my_cols >> (lane & 15) & 1u;
    uint32_t again = 0;                                                   // bit 4 m + v: this lane's output is computed again
#pragma unroll
    for (int m = 0; m < kSplitBlocks; ++m) {
        if (m >= blocks) break;
        const uint32_t small_rows = small[m] >> (4 * (lane >> 4));
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = 16 * m + 4 * (lane >> 4) + v;
            const size_t at = buffer_row(rm, min(r, rows - 1));
            const float u = acc[m][0][v], g = acc[m][NP - 1][v];
            if (r >= rows || col >= NC) continue;
            if (small_col || (small_rows >> v & 1u) || !in_range(u) || !in_range(g)) again |= 1u << (4 * m + v);
            C[at * NC + col] = UP ? u / (1.0f + expf(-u)) * g : u;
        }
    }

    // An operand that is infinite, or rounds to that, has no pieces that add up to it (it makes a NaN of all its sums), and
    // those of one below 2^-110 may fall short, which its partner may make any size: the outputs of such rows and columns once
    // more, and only these (a row's values are its own whatever the other rows of the tile are), on
    // the fp32 instruction.  A wavefront multiplies the blocks of 16 rows that hold some; a lane holds the four k
    // from 4 * (lane / 16) of every 16, and four partial sums share the reduction.  Layer of 2000 routes, d 1024, f 2816,
    // plain 315 to 360 us: one row of NaN 440, every row 1180 (one fused multiply-add after the other per lane took 18.5 and 26 ms).
#pragma unroll 1
    for (int m = 0; m < blocks; ++m) {
        const uint32_t mine = again >> (4 * m) & 15u;
        if (!__any(mine != 0)) continue;
        const float* a_row = A + (size_t)buffer_row(rm, min(16 * m + (lane & 15), rows - 1)) * K;
        struct Piece { float4 a[4]; float b[NP][4][4]; };
        auto fetch_plain = [&](int k0, Piece& q) {                        // 64 k; those past the end count as zero
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = k0 + 16 * j + kg / 2, at = min(k, K - 4);
                const bool in = k < K;
                const float4 t = *reinterpret_cast<const float4*>(a_row + at);
                q.a[j] = make_float4(in ? t.x : 0.f, in ? t.y : 0.f, in ? t.z : 0.f, in ? t.w : 0.f);
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const float4 w = *reinterpret_cast<const float4*>(Bbase + (size_t)p * d * f + (size_t)at * NC + 4u * b_col);
                    q.b[p][j][0] = in ? w.x : 0.f; q.b[p][j][1] = in ? w.y : 0.f; q.b[p][j][2] = in ? w.z : 0.f; q.b[p][j][3] = in ? w.w : 0.f;
                }
            }
        };
        f32x4 sum[4][NP];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int p = 0; p < NP; ++p) sum[j][p] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto multiply_plain = [&](const Piece& q) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        const float av[4] = {q.a[j].x, q.a[j].y, q.a[j].z, q.a[j].w};
                        sum[j][p] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], q.b[p][j][i], sum[j][p], 0, 0, 0);
                    }
        };
        Piece q0, q1;
        fetch_plain(0, q0);
#pragma unroll 1
        for (int k0 = 0; k0 < K; k0 += 128) {                             // past the end the last values are fetched again
            fetch_plain(k0 + 64, q1);
            __builtin_amdgcn_sched_barrier(0);
            multiply_plain(q0);
            __builtin_amdgcn_sched_barrier(0);
            fetch_plain(k0 + 128, q0);
            __builtin_amdgcn_sched_barrier(0);
            multiply_plain(q1);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const size_t at = buffer_row(rm, min(16 * m + 4 * (lane >> 4) + v, rows - 1));
            const float u = (sum[0][0][v] + sum[1][0][v]) + (sum[2][0][v] + sum[3][0][v]);
            const float g = (sum[0][NP - 1][v] + sum[1][NP - 1][v]) + (sum[2][NP - 1][v] + sum[3][NP - 1][v]);
            if (mine >> v & 1u) C[at * NC + col] = UP ? u / (1.0f + expf(-u)) * g : u;
        }
    }
}

int launch_ffn_f32(const float* a, int N, int d, int f, int E, const float* packed, const int32_t* counts,
                   const int32_t* starts, const int32_t* placement, int local_gpu, const int32_t* group_expert,
                   int n_weights, float* out, int32_t* plan, bool plan_ready, float* H, hipStream_t s) {
    int rc;
    if (!plan_ready) {
        PlanShape shape;
        if ((rc = ffn_plan_shape(MOE_F32, N, d, f, E, false, group_expert != nullptr, &shape)) != MOE_OK) return rc;
        // groups that may share an expert are merged; the row offsets of a merged bucket must fit 32 bits
        const bool mergeable = group_expert != nullptr && (size_t)N * (d > f ? d : f) < ((size_t)1 << 32);
        rc = launch_ffn_plan(counts, starts, placement, local_gpu, group_expert, n_weights, E, N, shape, mergeable, {}, plan, s);
        if (rc != MOE_OK) return rc;
    }
    const bool split = local_gpu < 0 && split_pays(N, d, f, E);
    const int tile_rows = split ? kF32SplitRows : kF32Tile, tile_cols = split ? kSplitCols : kF32Tile;
    const long long mt_max = (N + tile_rows - 1) / tile_rows + (E < N ? E : N);   // sum of ceil(n_e / tile_rows) never exceeds this
    // (the split kernel's two shares of an XCD are rounded up one by one)
    auto grid_for = [&](int columns) { return (mt_max * ((columns + tile_cols - 1) / tile_cols) + (split ? 2 : 1) * kF32Xcds - 1) / kF32Xcds * kF32Xcds; };
    const auto up = split ? &ffn_f32_split_kernel<true> : &ffn_f32_kernel<true>, down = split ? &ffn_f32_split_kernel<false> : &ffn_f32_kernel<false>;
    if (grid_for(f) > 0x7FFFFFFFll || grid_for(d) > 0x7FFFFFFFll)
        return fail(MOE_ERR_UNSUPPORTED, "moe_expert_ffn_grouped: too many tiles for one launch");
    {
        LaunchTimer timer(MOE_K_FFN_UP, s);
        hipLaunchKernelGGL(up, dim3((unsigned)grid_for(f)), dim3(256), 0, s, a, packed, d, f, H, plan);
        if ((rc = check_launch("moe_expert_ffn_grouped up launch")) != MOE_OK) return rc;
    }
    {
        LaunchTimer timer(MOE_K_FFN_DOWN, s);
        hipLaunchKernelGGL(down, dim3((unsigned)grid_for(d)), dim3(256), 0, s, (const float*)H, packed, d, f, out, plan);
        if ((rc = check_launch("moe_expert_ffn_grouped down launch")) != MOE_OK) return rc;
    }
    return MOE_OK;
}

}  // namespace moe
