// moe_receive_segments: the segment table of the buffer a GPU receives from the first all-to-all of an
// expert-parallel layer (paper Section 2.2 / Fig. 2b), built on the device from the ranks' gathered
// expert_counts so that no bucket size has to visit the host between dispatch and the expert FFN.
//
// Source rank s sends GPU `dest` its bucket for dest, already sorted by expert; the receive buffer is the
// concatenation of those buckets in source order.  Its segments are therefore, source after source, one run
// of rows per expert that lives on dest, experts ascending: segment (s, i-th expert of dest) holds
// expert_counts[s][e] rows.  The table feeds moe_expert_ffn_segments directly.
// The tables are tiny (at most 256 segments), so the call is one workgroup, bound by its rounds of memory and LDS latency:
// ranks and starts by ballots and scans; walking the tables in every thread, and with the plan that follows waiting for its stores,
// receives of 64 experts took 1 to 2.4 us longer (55.1 and 57.1, 99.1 and 101.5 us).
#include "common.h"

namespace moe {

__global__ __launch_bounds__(MOE_MAX_EXPERTS) void receive_segments_kernel(const int32_t* __restrict__ counts_all,
                                                                          const int32_t* __restrict__ placement, int E, int G, int dest,
                                                                          int max_seg, int32_t* __restrict__ seg_expert,
                                                                          int32_t* __restrict__ seg_counts, int32_t* __restrict__ seg_start,
                                                                          int32_t* __restrict__ src_offset, int32_t* __restrict__ n_seg_out) {
    constexpr int kWaves = MOE_MAX_EXPERTS / 64;
    __shared__ unsigned long long local_mask[kWaves];    // the experts of dest
    __shared__ int local_expert[MOE_MAX_EXPERTS];        // ... ascending
    __shared__ int wave_rows[kWaves];                    // rows of a wavefront's segments
    const int i = threadIdx.x, lane = i & 63, wave = i >> 6;
    const bool is_local = i < E && placement[i] == dest;
    const unsigned long long mine = __ballot(is_local);
    if (lane == 0) local_mask[wave] = mine;
    __syncthreads();
    int rank = __popcll(mine & ((1ull << lane) - 1ull)), n_local = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const int here = __popcll(local_mask[w]);
        rank += w < wave ? here : 0;
        n_local += here;
    }
    if (is_local) local_expert[rank] = i;
    __syncthreads();
    const long long wanted = (long long)G * n_local;
    const int n_seg = (int)(wanted < max_seg ? wanted : max_seg);
    int e = 0, c = 0, source = 0;
    if (i < n_seg) {
        source = i / n_local;
        e = local_expert[i - source * n_local];
        c = counts_all[(size_t)source * E + e];
        if (c < 0) c = 0;
    }
    int sum = c;                                         // of this wavefront's segments up to this one
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const int o = __shfl_up(sum, m, 64);
        sum += lane >= m ? o : 0;
    }
    if (lane == 63) wave_rows[wave] = sum;
    __syncthreads();
    int start = sum - c, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        start += w < wave ? wave_rows[w] : 0;
        total += wave_rows[w];
    }
    if (i < max_seg) {                                   // entries past the last segment are empty segments at the end of the buffer
        seg_expert[i] = e;
        seg_counts[i] = c;
        seg_start[i] = i < n_seg ? start : total;
    }
    if (src_offset != nullptr) {
        // source s begins at its first segment (s * n_local); sources whose segments did not fit, and the end, at the total
        if (i < n_seg && i == source * n_local) src_offset[source] = start;
        if (i < G && (long long)i * n_local >= n_seg) src_offset[i] = total;
        if (i == 0) src_offset[G] = total;
    }
    if (i == 0 && n_seg_out != nullptr) *n_seg_out = (int)(wanted < 0x7FFFFFFF ? wanted : 0x7FFFFFFF);
}

int launch_receive_segments(const int32_t* counts_all, const int32_t* placement, int E, int G, int dest, int max_seg,
                            int32_t* seg_expert, int32_t* seg_counts, int32_t* seg_start, int32_t* src_offset, int32_t* n_seg_out,
                            hipStream_t s) {
    hipLaunchKernelGGL(receive_segments_kernel, dim3(1), dim3(MOE_MAX_EXPERTS), 0, s, counts_all, placement, E, G, dest, max_seg,
                       seg_expert, seg_counts, seg_start, src_offset, n_seg_out);
    return check_launch("moe_receive_segments launch");
}

}  // namespace moe
