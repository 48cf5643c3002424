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
    int pl[MOE_MAX_EXPERTS];                  // the map; loaded by the caller before the barrier that precedes index_totals
    int tot[MOE_MAX_EXPERTS];                 // routes per expert
    int start[MOE_MAX_EXPERTS];               // first position of each expert
};

__device__ __forceinline__ void index_clear(IndexTables& s, int E) {
    for (int i = threadIdx.x; i < kIndexWaves * MOE_MAX_EXPERTS; i += kIndexThreads)
        if ((i & (MOE_MAX_EXPERTS - 1)) < E) (&s.woff[0][0])[i] = 0;
}

// Per-wavefront counts -> totals, expert starts and per-wavefront write offsets.  Called by all threads, after a
// barrier that follows the counting; ends with a barrier.
__device__ __forceinline__ void index_totals(IndexTables& s, int E) {
    const int me = threadIdx.x;
    if (me < E) {
        int t = 0;
#pragma unroll
        for (int w = 0; w < kIndexWaves; ++w) t += s.woff[w][me];
        s.tot[me] = t;
    }
    __syncthreads();
    if (me < E) {
        const int ge = s.pl[me];
        int start = 0;
#pragma unroll 8
        for (int o = 0; o < E; ++o) {
            const int go = s.pl[o];
            start += ((go < ge) | ((go == ge) & (o < me))) ? s.tot[o] : 0;
        }
        s.start[me] = start;
        int run = start;
#pragma unroll
        for (int w = 0; w < kIndexWaves; ++w) {
            const int c = s.woff[w][me];
            s.woff[w][me] = run;
            run += c;
        }
    }
    __syncthreads();
}

// expert_counts, expert_start and the per-GPU tables, from the totals; called by all threads after index_totals
__device__ __forceinline__ void index_write_tables(const IndexTables& s, int E, int G, int32_t* __restrict__ expert_counts,
                                                   int32_t* __restrict__ expert_start, int32_t* __restrict__ gpu_counts,
                                                   int32_t* __restrict__ gpu_offsets) {
    if ((int)threadIdx.x < E) {
        expert_counts[threadIdx.x] = s.tot[threadIdx.x];
        expert_start[threadIdx.x] = s.start[threadIdx.x];
    }
    for (int g = threadIdx.x; g < G; g += kIndexThreads) {
        int cnt = 0, off = 0;
#pragma unroll 8
        for (int o = 0; o < E; ++o) {
            const int go = s.pl[o], to = s.tot[o];
            cnt += (go == g) ? to : 0;
            off += ((go >= 0) & (go < g)) ? to : 0;
        }
        gpu_counts[g] = cnt;
        gpu_offsets[g] = off;
        if (g == G - 1) gpu_offsets[G] = off + cnt;
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

}  // namespace moe
