// The stable counting sort of moe_dispatch (paper Section 2.2, Section 3.1) done by ONE workgroup of 16 wavefronts,
// each owning a contiguous slice of the routes: shared by the dispatch index kernel and by the fused front of the
// layer.  Positions are a pure function of the route id.
#pragma once
#include "common.h"

namespace moe {

constexpr int kIndexThreads = 1024, kIndexWaves = kIndexThreads / 64;

// lanes of this wavefront that hold the same expert as the calling lane
__device__ __forceinline__ unsigned long long match_expert(int e, bool valid, int ebits) {
    unsigned long long m = __ballot(valid);
    for (int b = 0; b < ebits; ++b) {
        const bool bit = (e >> b) & 1;
        const unsigned long long v = __ballot(bit);
        m &= bit ? v : ~v;
    }
    return m;
}

struct IndexTables {
    int woff[kIndexWaves][MOE_MAX_EXPERTS];   // per wavefront: routes of each expert in its slice, then its next position
    int pl[MOE_MAX_EXPERTS];                  // the map; loaded by the caller before the barrier that precedes index_offsets
    int tot[MOE_MAX_EXPERTS];                 // routes per expert
    int start[MOE_MAX_EXPERTS];               // first position of each expert
};

__device__ __forceinline__ void index_clear(IndexTables& s, int E) {
    for (int i = threadIdx.x; i < kIndexWaves * MOE_MAX_EXPERTS; i += kIndexThreads)
        if ((i & (MOE_MAX_EXPERTS - 1)) < E) (&s.woff[0][0])[i] = 0;
    if ((int)threadIdx.x < E) s.start[threadIdx.x] = 0;
}

// Totals and per-wavefront counts -> expert starts and per-wavefront write offsets; `before` (in LDS, may be NULL):
// routes of each expert that precede this workgroup's.  Called by all threads, after a barrier; ends with one.
// The E x E comparisons of the starts are dealt to all threads (thread: expert, slice of the others), because one
// wavefront walking E = 64 totals took 3.7 us, more than the ranking of its routes.  The number of rounds is known before the
// loop, so that their reads overlap whatever the compiler makes of the code around (asked in every round whether there is
// a next, 2.1 us more at E = 256, where there are 64).
__device__ __forceinline__ void index_offsets(IndexTables& s, int E, int ebits, const int* before) {
    const int EP = 1 << ebits, me = threadIdx.x & (EP - 1), slices = kIndexThreads >> ebits;
    const int first = threadIdx.x >> ebits, rounds = (E << ebits) / kIndexThreads;   // in which every thread has an expert; one more in which some have
    int start = 0;
    if (me < E) {
        const int ge = s.pl[me];
        const auto before_me = [&](int o) {
            const int go = s.pl[o], to = s.tot[o];
            return (go < ge) | ((go == ge) & (o < me)) ? to : 0;
        };
#pragma unroll 4
        for (int i = 0; i < rounds; ++i) start += before_me(first + i * slices);
        if (first + rounds * slices < E) start += before_me(first + rounds * slices);
    }
    for (int m = EP; m < 64; m <<= 1) start += __shfl_xor(start, m, 64);
    if (me < E && (threadIdx.x & 63) < EP) atomicAdd(&s.start[me], start);          // cleared by index_clear
    __syncthreads();
    if ((int)threadIdx.x < E) {
        int run = s.start[me] + (before != nullptr ? before[me] : 0);
#pragma unroll
        for (int w = 0; w < kIndexWaves; ++w) {
            const int c = s.woff[w][me];
            s.woff[w][me] = run;
            run += c;
        }
    }
    __syncthreads();
}

// The same for a workgroup that counted every route itself: the totals are the sums of its wavefronts' counts.
__device__ __forceinline__ void index_totals(IndexTables& s, int E, int ebits) {
    const int me = threadIdx.x;
    if (me < E) {
        int t = 0;
#pragma unroll
        for (int w = 0; w < kIndexWaves; ++w) t += s.woff[w][me];
        s.tot[me] = t;
    }
    __syncthreads();
    index_offsets(s, E, ebits, nullptr);
}

// expert_counts, expert_start and the per-GPU tables, from the totals; called by all threads once the positions are
// out (it overwrites woff)
__device__ __forceinline__ void index_write_tables(IndexTables& s, int E, int G, int32_t* __restrict__ expert_counts,
                                                   int32_t* __restrict__ expert_start, int32_t* __restrict__ gpu_counts,
                                                   int32_t* __restrict__ gpu_offsets) {
    static_assert(MOE_MAX_GPUS <= MOE_MAX_EXPERTS, "the GPU tables are built in rows of woff");
    int* cnt = s.woff[0];
    int* off = s.woff[1];
    __syncthreads();
    if ((int)threadIdx.x < E) {
        expert_counts[threadIdx.x] = s.tot[threadIdx.x];
        expert_start[threadIdx.x] = s.start[threadIdx.x];
    }
    if ((int)threadIdx.x < G) cnt[threadIdx.x] = off[threadIdx.x] = 0;
    __syncthreads();
    int gbits = 0;
    while ((1 << gbits) < G) ++gbits;
    const int g = threadIdx.x & ((1 << gbits) - 1);
    if (g < G) {                                         // thread: GPU, slice of the experts
        int c = 0, f = 0;
        for (int o = threadIdx.x >> gbits; o < E; o += kIndexThreads >> gbits) {
            const int go = s.pl[o], to = s.tot[o];
            c += (go == g) ? to : 0;
            f += ((go >= 0) & (go < g)) ? to : 0;
        }
        if (c) atomicAdd(&cnt[g], c);
        if (f) atomicAdd(&off[g], f);
    }
    __syncthreads();
    if ((int)threadIdx.x < G) {
        gpu_counts[threadIdx.x] = cnt[threadIdx.x];
        gpu_offsets[threadIdx.x] = off[threadIdx.x];
        if ((int)threadIdx.x == G - 1) gpu_offsets[G] = off[threadIdx.x] + cnt[threadIdx.x];
    }
}

// the position of this lane's route (expert ex, valid when ok) among the wavefront's next 64; advances the wavefront's offsets
__device__ __forceinline__ int index_next(volatile int* my, int ex, bool ok, int ebits, unsigned long long lower) {
    const unsigned long long m = match_expert(ex, ok, ebits);
    int pos = 0;
    if (ok) pos = my[ex] + __popcll(m & lower);
    __builtin_amdgcn_wave_barrier();
    if (ok && (m & lower) == 0ull) my[ex] += __popcll(m);
    __builtin_amdgcn_wave_barrier();
    return pos;
}

// The same without LDS, for up to 64 experts (2^EB >= E): lane e keeps the wavefront's routes of expert e so far in `count`.
// Returns the rank of this lane's route among the wavefront's routes of its expert, and counts the 64 of this step.  A chain
// through LDS (index_next: read, write, wait, for every 64 routes) took 3.2 of the 13.4 us of ranking 2 M routes.
template <int EB>
__device__ __forceinline__ int wave_rank(int ex, bool ok, int& count) {
    static_assert(EB >= 1 && EB <= 6, "one lane per expert");
    const int lane = threadIdx.x & 63;
    const unsigned long long valid = __ballot(ok);
    uint32_t mine_lo = (uint32_t)valid, mine_hi = (uint32_t)(valid >> 32);     // lanes with this lane's expert
    uint32_t e_lo = mine_lo, e_hi = mine_hi;                                   // lanes with expert `lane`
#pragma unroll
    for (int b = 0; b < EB; ++b) {
        const unsigned long long v = __ballot((ex >> b) & 1);
        const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
        const uint32_t x = 0u - ((uint32_t)ex >> b & 1u), y = 0u - ((uint32_t)lane >> b & 1u);
        mine_lo &= ~(lo ^ x);
        mine_hi &= ~(hi ^ x);
        e_lo &= ~(lo ^ y);
        e_hi &= ~(hi ^ y);
    }
    const int before = __builtin_amdgcn_ds_bpermute((ex & 63) << 2, count);
    count += __popc(e_lo) + __popc(e_hi);                                      // lanes from E on count what nobody asks for
    return before + (int)__builtin_amdgcn_mbcnt_hi(mine_hi, __builtin_amdgcn_mbcnt_lo(mine_lo, 0u));
}

}  // namespace moe
