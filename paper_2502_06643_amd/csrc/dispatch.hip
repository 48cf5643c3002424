// moe_dispatch: placement-aware token dispatch (paper Section 1, Section 2.2,
// Section 3.1) as a stable counting sort of the N = T*k routes by the key
// (placement[expert], expert), followed by the row copy into the send buffer.
//
//   count : each workgroup histograms its contiguous chunk of routes by expert
//   rank  : each workgroup adds the histograms up (in total: expert_counts =
//           P_{e,l}; before its own chunk: where its routes begin), ranks the
//           experts by (gpu, expert) to get expert_start, and works out,
//           wavefront by wavefront, the stable rank of every route of its chunk
//           among the routes of the same expert (ballot match + popcount of the
//           lower lanes): perm / inv_perm.  One workgroup also writes the
//           expert and GPU tables
//   rows  : every 16-byte piece of x[t] is read once and written to the k
//           sorted positions of token t
//
// The result does not depend on how workgroups are scheduled: every position
// is a pure function of the route id.
#include <mutex>
#include "dispatch_index.h"
#include "ffn_late.h"

namespace moe {

constexpr int kMaxChunks = 1024;     // per-chunk histograms that a caller's workspace holds at most

// The workspace's geometry: what moe_dispatch_workspace_bytes promises room for.  The kernels below use
// chunks of at least this size (route_chunks), so their histograms always fit.
void dispatch_geometry(long long N, int* items, int* nblocks) {
    long long it = (N + (long long)kMaxChunks * kDispatchBlock - 1) / ((long long)kMaxChunks * kDispatchBlock);
    if (it < kDispatchItems) it = kDispatchItems;
    it = (it + 3) / 4 * 4;
    *items = (int)it;
    *nblocks = (int)((N + it * kDispatchBlock - 1) / (it * kDispatchBlock));
}

// A chunk is what one workgroup of 16 wavefronts counts and ranks: 1024 routes times `steps`.  At most
// kRankChunks chunks, one per compute unit: every rank workgroup reads all their histograms.
constexpr int kRankChunks = 256;         // 512: the same at E = 8, 12.2 against 8.7 us at E = 64
static void route_chunks(long long N, int* steps, int* chunks) {
    const long long st = (N + (long long)kRankChunks * kIndexThreads - 1) / ((long long)kRankChunks * kIndexThreads);
    *steps = (int)st;
    *chunks = (int)((N + st * kIndexThreads - 1) / (st * kIndexThreads));
}

constexpr int kCountCopies = 256;        // LDS counters of a workgroup
static_assert(kCountCopies >= MOE_MAX_EXPERTS && kCountCopies <= kIndexThreads, "a thread per counter");
// MANY: several copies of the histogram, picked by lane, because the lanes that hold the same expert queue on one address.  For few
// experts and several steps a workgroup (8 experts, 2 M routes: 5.4 us with one copy, 4.0 with 32; 40000 routes 2.7 and 3.2; 64
// experts, 600 k routes: 3.1 with one, 3.4 with 4, 4.0 with 32)
template <bool MANY>
__global__ __launch_bounds__(kIndexThreads) void dispatch_count_kernel(const int32_t* __restrict__ topk_idx, int N, int E, int steps, int copies,
                                                                       int32_t* __restrict__ block_counts) {
    __shared__ int hist[kCountCopies];
    const int copy = threadIdx.x & (copies - 1);
    if ((int)threadIdx.x < (MANY ? kCountCopies : E)) hist[threadIdx.x] = 0;
    __syncthreads();
    const long long base = (long long)blockIdx.x * kIndexThreads * steps + threadIdx.x;
    for (int i0 = 0; i0 < steps; i0 += 8) {
        int e[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const long long r = base + (long long)(i0 + u) * kIndexThreads;
            e[u] = (i0 + u < steps && r < N) ? topk_idx[r] : -1;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if ((unsigned)e[u] < (unsigned)E) atomicAdd(&hist[MANY ? e[u] * copies + copy : e[u]], 1);
    }
    __syncthreads();
    const int i = threadIdx.x;
    if (!MANY) {
        if (i < E) block_counts[(size_t)blockIdx.x * E + i] = hist[i];
    } else if (i < kCountCopies) {                       // whole wavefronts: adjacent lanes add up the copies of one expert
        int c = i < E * copies ? hist[i] : 0;
        for (int m = 1; m < copies; m <<= 1) c += __shfl_xor(c, m, 64);
        if (i < E * copies && (i & (copies - 1)) == 0) block_counts[(size_t)blockIdx.x * E + i / copies] = c;
    }
}

// the tile plan of the expert FFN, by a workgroup that holds the totals and starts (all threads call this)
__device__ __forceinline__ void plan_from_tables(const IndexTables& s, PlanScratch& scratch, int E, const PlanTask& pt) {
    const int e = threadIdx.x;
    int c = 0, st = 0;
    if (e < E && (pt.local_gpu < 0 || s.pl[e] == pt.local_gpu)) {
        c = s.tot[e];
        st = s.start[e];
    }
    build_plan(scratch, e, c, st, e, E, pt.shape, pt.plan, false, 0, pt.late.T > 0);
}

// Ranks the routes of one chunk.  Latency-bound: every workgroup adds up all chunks' histograms for itself
// (at most kRankChunks x E counts, L2 hits, independent loads) instead of waiting for a scan kernel of one
// workgroup, whose two dependent walks over up to 1024 histograms took 22 us at E = 64 (600 k routes; count, scan
// and rank 34 us, count and rank now 11.2 us) and 6.6 us at E = 8 (2 M routes: 25 -> 13.4 us).  Of the 10.7 us of the rank
// kernel for 2 M routes the ranks are 1.5 (wave_rank; with the histograms read before them and a chain through LDS 12.4;
// 64 experts, 600 k routes 9.5, 9.2 in lanes), the scattered stores 1.5, the rest launch, loads and barriers.
// The workgroup of the first chunk also writes the tables; a tile plan is written by one more, which comes first.
constexpr int kRankBatch = 8;            // 64-route steps of a wavefront whose expert ids are in registers together
// EB: bits of an expert id, for wave_rank; 0: counted in LDS.  HIST: histogram entries of a thread in flight together; up to 256 chunks
// over 1024 / 8, 16, 32 or 64 slices make 2, 4, 8 or 16 of them.
template <int EB, int HIST>
__global__ __launch_bounds__(kIndexThreads) void dispatch_rank_kernel(const int32_t* __restrict__ topk_idx, int N, int E, int ebits, int steps,
                                                                      const int32_t* __restrict__ block_counts,
                                                                      const int32_t* __restrict__ placement, int G,
                                                                      int32_t* __restrict__ expert_counts,
                                                                      int32_t* __restrict__ expert_start,
                                                                      int32_t* __restrict__ gpu_counts,
                                                                      int32_t* __restrict__ gpu_offsets,
                                                                      int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm,
                                                                      PlanTask pt) {
    __shared__ IndexTables s;
    __shared__ PlanScratch plan_scratch;
    __shared__ int before[MOE_MAX_EXPERTS];              // routes of each expert in the chunks before this one
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int extra = pt.plan != nullptr ? 1 : 0, chunks = (int)gridDim.x - extra, chunk = (int)blockIdx.x - extra;
    const long long wbase = chunk < 0 ? N : ((long long)chunk * kIndexWaves + wave) * 64 * steps;
    const unsigned long long lower = (1ull << lane) - 1ull;
    int exs[kRankBatch], loc[kRankBatch];                // expert of a route, its rank among the wavefront's routes of that expert
    auto load = [&](int i0) {
#pragma unroll
        for (int u = 0; u < kRankBatch; ++u) {
            const long long r = wbase + (long long)(i0 + u) * 64 + lane;
            exs[u] = (i0 + u < steps && r < N) ? topk_idx[r] : -1;
        }
    };
    // all chunks' histograms: thread (expert, slice of the chunks), then the slices of a wavefront, then LDS.  Where the ranks
    // are counted in lanes the first entries are asked for before the routes are ranked and added up after that; where
    // both go through LDS the histograms come first (128 experts, 600 k routes 12.8 us for 12.2 the other way round)
    const int EP = 1 << ebits, he = threadIdx.x & (EP - 1), slices = kIndexThreads >> ebits;
    int first[HIST], all = 0, mine = 0;
    auto fetch = [&](int b0, int (&c)[HIST]) {
#pragma unroll
        for (int u = 0; u < HIST; ++u) {
            const int b = b0 + u * slices;
            c[u] = he < E && b < chunks ? block_counts[(size_t)b * E + he] : 0;
        }
    };
    auto add = [&](int b0, const int (&c)[HIST]) {
#pragma unroll
        for (int u = 0; u < HIST; ++u) {
            all += c[u];
            mine += b0 + u * slices < chunk ? c[u] : 0;
        }
    };
    int b0 = threadIdx.x >> ebits;
    auto histograms = [&]() {
        if (he < E) {
            for (; b0 < chunks; b0 += HIST * slices) {
                int c[HIST];
                fetch(b0, c);
                add(b0, c);
            }
        }
        for (int m = EP; m < 64; m <<= 1) {
            all += __shfl_xor(all, m, 64);
            mine += __shfl_xor(mine, m, 64);
        }
        if (he < E && lane < EP) {
            atomicAdd(&s.tot[he], all);
            atomicAdd(&before[he], mine);
        }
    };
    load(0);
    if (EB > 0) fetch(b0, first);
    index_clear(s, E);
    if ((int)threadIdx.x < E) {
        s.pl[threadIdx.x] = placement[threadIdx.x];
        s.tot[threadIdx.x] = 0;
        before[threadIdx.x] = 0;
    }
    __syncthreads();

    if (EB == 0) histograms();
    // this wavefront's own routes are counted and ranked in one go;
    // the ranks stay in registers, those of a slice of more than kRankBatch steps wait in inv_perm
    const bool spill = steps > kRankBatch;
    int count = 0;
    for (int i0 = 0;;) {
#pragma unroll
        for (int u = 0; u < kRankBatch; ++u) {
            loc[u] = 0;
            if (i0 + u >= steps) continue;
            const bool ok = (unsigned)exs[u] < (unsigned)E;
            if constexpr (EB > 0) loc[u] = wave_rank<EB>(exs[u], ok, count);
            else loc[u] = index_next(s.woff[wave], exs[u], ok, ebits, lower);     // a wavefront's LDS accesses execute in order
            if (spill && ok) inv_perm[wbase + (long long)(i0 + u) * 64 + lane] = loc[u];
        }
        i0 += kRankBatch;
        if (i0 >= steps) break;
        load(i0);
    }
    if (EB > 0) {
        if (lane < E) s.woff[wave][lane] = count;
        add(b0, first);
        b0 += HIST * slices;
        histograms();
    }
    __syncthreads();
    index_offsets(s, E, ebits, before);

    for (int i0 = 0; i0 < steps; i0 += kRankBatch) {
        if (spill) {
            load(i0);
#pragma unroll
            for (int u = 0; u < kRankBatch; ++u)
                if ((unsigned)exs[u] < (unsigned)E) loc[u] = inv_perm[wbase + (long long)(i0 + u) * 64 + lane];
        }
#pragma unroll
        for (int u = 0; u < kRankBatch; ++u) {
            if ((unsigned)exs[u] >= (unsigned)E) continue;
            const long long r = wbase + (long long)(i0 + u) * 64 + lane;
            const int pos = s.woff[wave][exs[u]] + loc[u];
            perm[pos] = (int32_t)r;
            inv_perm[r] = pos;
        }
    }
    if (chunk < 0) plan_from_tables(s, plan_scratch, E, pt);
    else if (chunk == 0) index_write_tables(s, E, G, expert_counts, expert_start, gpu_counts, gpu_offsets);
}

// Batches of up to kFusedMaxRoutes routes: count and rank in ONE workgroup of 16 wavefronts, each
// owning a contiguous slice of the routes.  Two launches become one, which is what matters at these
// sizes (every launch costs more than the work it does).  A thread keeps its ITEMS expert ids in
// registers: they are loaded once, all loads in flight together, and serve both passes.  Same
// results: positions are a pure function of the route id.
constexpr int kFusedMaxItems = 16;
constexpr int kFusedMaxRoutes = kIndexThreads * kFusedMaxItems;

template <int ITEMS>
__global__ __launch_bounds__(kIndexThreads) void dispatch_index_kernel(const int32_t* __restrict__ topk_idx, int N, int E, int ebits,
                                                                       const int32_t* __restrict__ placement, int G,
                                                                       int32_t* __restrict__ expert_counts,
                                                                       int32_t* __restrict__ expert_start,
                                                                       int32_t* __restrict__ gpu_counts,
                                                                       int32_t* __restrict__ gpu_offsets,
                                                                       int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm,
                                                                       PlanTask pt) {
    __shared__ IndexTables s;
    __shared__ PlanScratch plan_scratch;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    index_clear(s, E);
    if ((int)threadIdx.x < E) s.pl[threadIdx.x] = placement[threadIdx.x];
    __syncthreads();

    const int wbase = wave * ITEMS * 64;                                // ITEMS 64-route steps per wavefront
    const unsigned long long lower = (1ull << lane) - 1ull;
    int exs[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int r = wbase + i * 64 + lane;
        exs[i] = (r < N) ? topk_idx[r] : -1;
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if ((unsigned)exs[i] < (unsigned)E) atomicAdd(&s.woff[wave][exs[i]], 1);   // LDS atomics: counts need no order
    __syncthreads();
    index_totals(s, E, ebits);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int r = wbase + i * 64 + lane;
        const bool ok = (unsigned)exs[i] < (unsigned)E;
        const int pos = index_next(s.woff[wave], exs[i], ok, ebits, lower);
        if (ok) {
            perm[pos] = (int32_t)r;
            inv_perm[r] = pos;
        }
    }
    index_write_tables(s, E, G, expert_counts, expert_start, gpu_counts, gpu_offsets);
    if (pt.plan != nullptr) plan_from_tables(s, plan_scratch, E, pt);
}

// One thread per 16-byte unit of a source row: read once, write k times.  LATE: of the first tokens only the rows of this
// GPU's experts; the projections copy the others (ffn_late.h), and read in the plan's header how many tokens that are.  This GPU's
// rows follow each other in the sorted order, so they are looked up there, and what is read of x is what is copied.
// Bound by three rounds of memory latency: 8192 tokens, 64 experts, top-6, 8 of them here, d 2048: 9.4 us, layer 139; walking the
// tokens and reading all of x 14.4 and 143.
template <bool LATE>
__global__ __launch_bounds__(256) void dispatch_rows_kernel(const uint4* __restrict__ x, long long total_units, int units_per_row,
                                                            int k, int N, const int32_t* __restrict__ perm, const int32_t* __restrict__ inv_perm,
                                                            uint4* __restrict__ send_buf, LateShape late, const int32_t* __restrict__ plan,
                                                            int32_t* __restrict__ plan_late) {
    const long long u = (long long)blockIdx.x * 256 + threadIdx.x;
    if (u >= total_units) return;
    long long t = u / units_per_row;
    const int c = (int)(u - t * units_per_row);
    if (LATE) {
        const int own0 = plan[kPlanOwnBegin], own1 = plan[kPlanOwnEnd];
        const LateTokens n = late_tokens(late, plan, own1 - own0);
        if (u == 0) {
            plan_late[0] = n.up;
            plan_late[1] = n.down;
        }
        const int late_here = n.up + n.down, place = (int)t - (late.T - late_here);
        if (place >= 0) {                                // as many places as there are late tokens
            for (int p = own0 + place; p < own1; p += late_here) {
                const int of = perm[p] / k;
                if (of < late_here) send_buf[(long long)p * units_per_row + c] = x[(long long)of * units_per_row + c];
            }
            return;
        }
        t += late_here;
    }
    const uint4 v = x[t * units_per_row + c];
    for (int j = 0; j < k; ++j) {
        const int p = inv_perm[t * k + j];
        if (p >= 0 && p < N) send_buf[(long long)p * units_per_row + c] = v;
    }
}

// Scratch of moe_dispatch_noalloc: the per-chunk expert histograms (count -> rank) in device memory
// that exists from the moment the library is loaded, so that the call allocates nothing.  Every GPU the
// library runs on holds its own copy at its own address; in host code the array's name is only a handle
// for hipGetSymbolAddress, never a pointer to pass to a kernel.  The count kernel writes every entry the
// rank kernel reads, so nothing has to be cleared between calls; calls that overlap on one GPU
// share the array and race.
static __device__ __align__(256) unsigned char dispatch_scratch[kDispatchStaticScratchBytes];

constexpr int kMaxDevices = 64;

int dispatch_static_scratch(int32_t** scratch) {
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "moe_dispatch_noalloc: hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(MOE_ERR_UNSUPPORTED, "moe_dispatch_noalloc: device %d outside [0,%d)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(mu);
    if (addr[dev] == nullptr) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(dispatch_scratch));     // this device's copy (dev is current)
        if (e != hipSuccess) return hip_fail(e, "moe_dispatch_noalloc: hipGetSymbolAddress");
        if (p == nullptr) return fail(MOE_ERR_HIP, "moe_dispatch_noalloc: no device address for the scratch array");
        addr[dev] = p;
    }
    *scratch = static_cast<int32_t*>(addr[dev]);
    return MOE_OK;
}

int launch_dispatch(const void* x, int row_bytes, const int32_t* topk_idx, int T, int E, int k,
                    const int32_t* placement, int G, void* send_buf, int32_t* perm, int32_t* inv_perm,
                    int32_t* expert_counts, int32_t* expert_start, int32_t* gpu_counts,
                    int32_t* gpu_offsets, int32_t* block_counts, const PlanTask& plan_task, hipStream_t s) {
    const int N = T * k;
    int ebits = 0;
    while ((1 << ebits) < E) ++ebits;
    int rc;
    if (N <= kFusedMaxRoutes) {
        LaunchTimer timer(MOE_K_DISPATCH_RANK, s);
#define MOE_LAUNCH_INDEX(ITEMS)                                                                                          \
    hipLaunchKernelGGL(dispatch_index_kernel<ITEMS>, dim3(1), dim3(kIndexThreads), 0, s, topk_idx, N, E, ebits, placement, G, \
                       expert_counts, expert_start, gpu_counts, gpu_offsets, perm, inv_perm, plan_task)
        if (N <= kIndexThreads) MOE_LAUNCH_INDEX(1);
        else if (N <= 2 * kIndexThreads) MOE_LAUNCH_INDEX(2);
        else if (N <= 4 * kIndexThreads) MOE_LAUNCH_INDEX(4);
        else if (N <= 8 * kIndexThreads) MOE_LAUNCH_INDEX(8);
        else MOE_LAUNCH_INDEX(kFusedMaxItems);
#undef MOE_LAUNCH_INDEX
        if ((rc = check_launch("moe_dispatch index launch")) != MOE_OK) return rc;
    } else {
        int steps, chunks;
        route_chunks(N, &steps, &chunks);
        {
            LaunchTimer timer(MOE_K_DISPATCH_COUNT, s);
            int copies = 32;                             // a power of two
            while (E * copies > kCountCopies) copies /= 2;
            const bool many = E <= 32 && steps > 1;
            hipLaunchKernelGGL(many ? &dispatch_count_kernel<true> : &dispatch_count_kernel<false>, dim3(chunks), dim3(kIndexThreads), 0, s,
                               topk_idx, N, E, steps, copies, block_counts);
            if ((rc = check_launch("moe_dispatch count launch")) != MOE_OK) return rc;
        }
        {
            LaunchTimer timer(MOE_K_DISPATCH_RANK, s);
            // Counted in LDS: one step a wavefront (up to 262144 routes), as one count does not queue and the code is short
            // (8 experts, 16400 routes: dispatch 7.5 us, 8.2 in lanes; 64 experts, 131070 routes 8.5, 8.7); and more than 16 experts
            // where there are more workgroups than compute units, a layer call's 256 chunks and the plan (131072 tokens, 32 experts,
            // top-4: rank 8.8 us, 10.2 in lanes), as those in lanes have too many registers for two on a compute unit: 65 with 8
            // histogram entries, 81 with 16.  Up to 16 experts 50 and 54 (262144 tokens, 8 experts, top-2: 8.4 us; 9.8 with 76)
            const int groups = chunks + (plan_task.plan != nullptr ? 1 : 0);
            const auto rank = steps == 1 || ebits > 6 || (ebits > 4 && groups > kRankChunks) ? &dispatch_rank_kernel<0, 16>
                              : ebits <= 3 ? &dispatch_rank_kernel<3, 2> : ebits <= 4 ? &dispatch_rank_kernel<4, 4>
                              : ebits <= 5 ? &dispatch_rank_kernel<6, 8> : &dispatch_rank_kernel<6, 16>;
            hipLaunchKernelGGL(rank, dim3(groups), dim3(kIndexThreads), 0, s, topk_idx, N, E, ebits, steps, block_counts,
                               placement, G, expert_counts, expert_start, gpu_counts, gpu_offsets, perm, inv_perm, plan_task);
            if ((rc = check_launch("moe_dispatch rank launch")) != MOE_OK) return rc;
        }
    }
    if (x != nullptr && N > 0) {
        const int units_per_row = row_bytes / 16;
        const long long total_units = (long long)T * units_per_row;
        const long long grid = (total_units + 255) / 256;
        if (grid > 0x7FFFFFFFll) return fail(MOE_ERR_UNSUPPORTED, "moe_dispatch: T*d too large for one launch");
        LaunchTimer timer(MOE_K_DISPATCH_ROWS, s);
        const auto rows = plan_task.late.T > 0 ? &dispatch_rows_kernel<true> : &dispatch_rows_kernel<false>;
        hipLaunchKernelGGL(rows, dim3((unsigned)grid), dim3(256), 0, s, (const uint4*)x, total_units,
                           units_per_row, k, N, perm, inv_perm, (uint4*)send_buf, plan_task.late, plan_task.plan,
                           plan_task.plan != nullptr ? plan_task.plan + kPlanLateUp : nullptr);
        if ((rc = check_launch("moe_dispatch rows launch")) != MOE_OK) return rc;
    }
    return MOE_OK;
}

}  // namespace moe
